// The up-projection, and the stage without dedicated consumers (included by
// moe_gemm2.hip, inside its anonymous namespace, after its helpers): a grouped
// GEMM with tiles that follow the batch, then a launch that combines, one wave
// per token and 256 or 512 columns.  The kernel boundary is the only
// dependency: no flags, no waits, nothing that has to be resident.  (The two
// launches run back to back on the GPU: no gap in a kernel trace.)
//
// What bounds such a launch: below about 64 rows per expert the weights (W2
// of 32 experts at H = 2048, I = 704 is 92 MB, 18.6 us at the rate a large
// copy reaches here), above it the tiles' operand traffic and the matrix
// cores.  The persistent kernel's 256 x 256 tiles give a workgroup 16-20 us of
// work whatever the rows in them, and its publish, readiness and acquire
// another 10-15 us.  Small tiles, one workgroup each and two or three per CU,
// let one's loads cover another's start, epilogue and waits; large batches
// run full tiles and give the small ones the rest (mixed_gemm_kernel).
//
// Every output element is the same chain as in the persistent kernel: the
// same 32x32x16 MFMAs over the whole reduction in the same order, Y rounded
// once to bf16, the rows of a token summed in ascending order.  So a
// reduction is never split over waves, and the results are bitwise equal.
//
// Measured (us a call, two sets of inputs in turn, persistent kernel -> this
// path), H = 2048, I = 704, E = 32, top-6, uniform routing: T = 64 42.3 -> 20.6,
// 256 45.6 -> 21.9, 512 49.4 -> 27.5, 1024 56.5 -> 38.8, 2048 81.6 -> 70.2, 4096
// 128 -> 118, 8192 237 -> 202, 16384 426 -> 389, 32768 789 -> 763 (T = 1, GPU time
// alone, 36.7 -> 9.8); its up-projection T = 64 59.7 -> 39.0, 256 60.5 -> 41.6, 512
// 62.6 -> 49.4, 1024 67.1 / 68.9, 2048 117 -> 105, 4096 174 -> 161, 8192 293 ->
// 284, 16384 567 -> 535.  The largest GEMMs are bound by the power the chip may
// draw: the up-projection of T = 16384 takes 515 us on one set of random operands
// and 396 us on zeros.
#pragma once

// A tile of BM rows x BN columns, its NW waves WNW along the columns, a ring
// of S stages of BK reduction steps in LDS (S - 1 of them in flight).  (32
// steps, half lines of x, let two 128 x 256 tiles of eight waves share a CU:
// four waves per SIMD and three quarters of the operand traffic of 128 x 128
// tiles.  Sixteen waves on a 256 x 256 tile, or four on a 128 x 256 one,
// measured slower: 123.9 and 155 against 118.9 us at T = 4096.)

template <int BM_, int BN_, int NW_, int WNW_, int S_, int BK_ = kBK>
struct SmallTile {
  static constexpr int BK = BK_, KS = BK / 16, XC = BK / 8;   // x chunks per row
  static constexpr int kXPerLine = 256 / (2 * BK);
  static constexpr int BM = BM_, BN = BN_, NW = NW_, WNW = WNW_, S = S_;
  static constexpr int WMW = NW / WNW;
  static constexpr int WN = BN / WNW, WM = BM / WMW;   // a wave's columns and rows
  static constexpr int NB = WN / 32, MB = WM / 32;
  static constexpr int kThr = NW * 64;
  static constexpr int XL = BM * BK / 512 / NW;   // 1 KB loads per wave and stage
  static constexpr int WL = BN * BK / 512 / NW;
  static constexpr int LPS = XL + WL;
  static constexpr int kXElems = BM * BK, kWElems = BN * BK;
  static constexpr int kSlot = kXElems + kWElems;
  static constexpr int WC = BN / 8;       // 16-byte chunks per W row
  static_assert(BN >= 64 && BN <= 512 && XL >= 1 && WL >= 1, "loads per wave");
  static_assert((S - 2) * LPS <= 63, "vmcnt range");
  // chunk swizzle of W row k: the 4 rows x 64 bytes one transposing read
  // touches fall on distinct banks
  static __device__ __forceinline__ int wswz(int k) { return BN == 64 ? 4 * ((k >> 1) & 1) : 4 * (k & 3); }
};

// a lane's global addresses for its loads of a tile's stages
template <class C>
struct SmallCtx {
  i32x4 ra, rb;
  uint32_t xo[C::XL], wo[C::WL];
  int xk[C::XL], wk[C::WL];
  uint32_t lds;
};

// Stage kt's loads into ring slot `slot`.  Stages past the reduction are
// issued as well (out of range: zeros, no memory request), so that every
// stage adds LPS to vmcnt.
template <class C, class Args>
__device__ __forceinline__ void small_issue(const Args& a, const SmallCtx<C>& t, int kt, int slot,
                                            int wave) {
  const int k0 = kt * C::BK;
  const uint32_t base = t.lds + (uint32_t)slot * (C::kSlot * 2);
#pragma unroll
  for (int q = 0; q < C::WL; ++q) {
    const int kw = k0 + t.wk[q];
    dma16(t.rb, kw < gemm_k(a) ? t.wo[q] + 2u * (uint32_t)k0 * (uint32_t)gemm_ldb(a) : kOutOfRange,
          base + (uint32_t)(C::kXElems * 2 + (C::WL * wave + q) * 1024));
  }
#pragma unroll
  for (int q = 0; q < C::XL; ++q) {
    const int kx = k0 + t.xk[q];
    dma16(t.ra, kx < gemm_k(a) ? t.xo[q] + 2u * (uint32_t)k0 : kOutOfRange,
          base + (uint32_t)((C::XL * wave + q) * 1024));
  }
}

// byte offset of the A row `row` of the tile at r0
__device__ __forceinline__ uint32_t small_a_off(const KArgs& a, int r0, int row) {
  return (uint32_t)row * (uint32_t)a.I * 2u;
}
__device__ __forceinline__ uint32_t small_a_off(const G1Args& a, int r0, int row) {
  int t = a.token_ids[(long long)r0 + row];
  if (t < 0 || t >= a.T) {
    __hip_atomic_fetch_or(a.status, kStBadRouting, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    t = 0;
  }
  return (uint32_t)t * (uint32_t)a.H * 2u;
}
__device__ __forceinline__ int small_n(const KArgs& a) { return a.H; }
__device__ __forceinline__ int small_n(const G1Args& a) { return 2 * a.I; }

// The rows of 64 K experts from e0 on, K neighbouring ones in each lane, by one
// round trip (with K = 1 alone, E = 1024 experts took a wave 16 of them for each
// tile: the stage of H = 1024, I = 256, 16 rows each 316 us, now 151).  Clamped as
// in load_experts; experts past E are empty.
template <int K>
struct ExpertRows {
  int start[K], count[K];
  bool bad;   // this lane's offsets are not a non-decreasing prefix of [0, rows]
  __device__ __forceinline__ ExpertRows(const int32_t* offsets, long long rows, int E, int e0) {
    const int e = e0 + K * (threadIdx.x & 63), cap = (int)rows;
    int off[K + 1];
#pragma unroll
    for (int i = 0; i <= K; ++i) off[i] = offsets[min(e + i, E)];
    bad = e == 0 && off[0] != 0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      bad |= off[i + 1] < off[i] || off[i + 1] > cap;
      start[i] = min(max(off[i], 0), cap);
      count[i] = max(min(off[i + 1], cap) - start[i], 0);   // (experts past E: off[i + 1] is off[i])
    }
  }
  template <class Units>
  __device__ __forceinline__ int sum(Units units) const {   // of this lane's experts
    int n = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) n += units(count[i]);
    return n;
  }
};

// An expert's rows, its first m-unit and how many it has.
struct ExpertUnit {
  int e, start, count, first, n;
};
// The expert that holds m-unit mt of the chunk at e0, which starts at m-unit
// `carry`; v: the inclusive prefix of the lanes' sums.
template <int K, class Units>
__device__ __forceinline__ ExpertUnit find_expert(const ExpertRows<K>& r, int e0, int mt, Units units,
                                                  int carry, int v) {
  // the first lane whose prefix passes mt, and its expert that does
  const int l = (int)__builtin_ctzll(__ballot(carry + v > mt));
  int k = 0, first = carry + v - r.sum(units), start = r.start[0], count = r.count[0], n = units(count);
#pragma unroll
  for (int i = 1; i < K; ++i)
    if (mt >= first + n) {
      first += n;
      k = i, start = r.start[i], count = r.count[i], n = units(count);
    }
  return {e0 + K * l + __builtin_amdgcn_readlane(k, l), __builtin_amdgcn_readlane(start, l),
          __builtin_amdgcn_readlane(count, l), __builtin_amdgcn_readlane(first, l),
          __builtin_amdgcn_readlane(n, l)};
}

__device__ __forceinline__ int wave_prefix(int v) {   // inclusive, over the lanes
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(v, d);
    if (lane >= d) v += u;
  }
  return v;
}

struct SmallUnit {
  int e, r0, rows_valid, n0;
  bool ok;
};

// This workgroup's unit (expert -> n-tile -> m-tile; consecutive units of an
// XCD are neighbours), by each wave for itself.
template <int BM, int BN, int K>
__device__ __forceinline__ SmallUnit small_unit_of(const int32_t* offsets, long long rows, int E, int NT,
                                                   uint32_t* status, int* rows_dev) {
  constexpr int kChunk = 64 * K;
  auto tiles = [](int count) { return (count + BM - 1) / BM; };
  ExpertRows<K> r(offsets, rows, E, 0);
  bool bad = r.bad;
  int mine = r.sum(tiles), e0 = 0;
  for (int e = kChunk; e < E; e += kChunk) {   // (the last chunk stays in r)
    r = ExpertRows<K>(offsets, rows, E, e0 = e);
    bad |= r.bad;
    mine += r.sum(tiles);
  }
  // the last row: the end of the last lane's last expert, empty or not
  *rows_dev = __builtin_amdgcn_readlane(r.start[K - 1] + r.count[K - 1], 63);
  if (bad && blockIdx.x == 0)
    __hip_atomic_fetch_or(status, kStBadRouting, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int v = wave_prefix(mine);
  SmallUnit u = {0, 0, 0, 0, false};
  const int b = blockIdx.x;
  const long long units = (long long)__builtin_amdgcn_readlane(v, 63) * NT;
  const long long chunk = (units + 7) >> 3;
  const long long unit = (long long)(b & 7) * chunk + (b >> 3);
  u.ok = (b >> 3) < chunk && unit < units;
  if (!u.ok) return u;
  const int mt = (int)(unit / NT);
  int carry = 0;
  if (E > kChunk) {
    for (e0 = 0;; e0 += kChunk) {
      r = ExpertRows<K>(offsets, rows, E, e0);
      v = wave_prefix(r.sum(tiles));
      const int sum = __builtin_amdgcn_readlane(v, 63);
      if (mt < carry + sum) break;
      carry += sum;
      u.ok = e0 + kChunk < E;   // (always: mt is below their sum)
      if (!u.ok) return u;
    }
  }
  const ExpertUnit x = find_expert(r, e0, mt, tiles, carry, v);
  const int within = (int)(unit - (long long)x.first * NT);
  const int nt = within / x.n;
  const int mi = within - nt * x.n;
  u.e = x.e;
  u.n0 = nt * BN;
  u.r0 = x.start + mi * BM;
  u.rows_valid = min(BM, x.count - mi * BM);
  return u;
}
template <int BM, int BN>
__device__ __forceinline__ SmallUnit small_unit(const int32_t* offsets, long long rows, int E, int NT,
                                                uint32_t* status, int* rows_dev) {
  return E <= 64    ? small_unit_of<BM, BN, 1>(offsets, rows, E, NT, status, rows_dev)
         : E <= 128 ? small_unit_of<BM, BN, 2>(offsets, rows, E, NT, status, rows_dev)
                    : small_unit_of<BM, BN, 4>(offsets, rows, E, NT, status, rows_dev);
}

// The tile's Y rows, through each wave's own part of the ring to 64- or
// 128-byte row pieces (as the persistent kernel's epilogue).
template <class C>
__device__ __forceinline__ void small_store(const KArgs& a, f32x16 (&acc)[C::NB][C::MB],
                                            uint16_t* smem, const SmallUnit& u, int wave, int lane,
                                            int wn0, int wm0, int n0, int cols_valid) {
  constexpr int EC = C::WN / 8;
  constexpr int kPerLine = 256 / (2 * C::WN);
  const int h = lane >> 5;
  __attribute__((address_space(3))) uint16_t* ep =
      (__attribute__((address_space(3))) uint16_t*)(uintptr_t)lds_addr(smem) + wave * (C::WM * C::WN);
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb) {
    const int row = 32 * mb + (lane & 31);
    const int sw = (row / kPerLine) % EC;
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        bf16x8 v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (__bf16)acc[nb][mb][8 * c + i];
        const int chunk = 4 * nb + 2 * c + h;
        *(__attribute__((address_space(3))) bf16x8*)(ep + row * C::WN + ((chunk ^ sw) << 3)) = v;
      }
  }
  const int j = lane % EC;
  const int n = wn0 + 8 * j;
#pragma unroll
  for (int it = 0; it < C::WM * EC / 64; ++it) {
    const int row = it * (64 / EC) + lane / EC;
    const int sw = (row / kPerLine) % EC;
    const bf16x8 v =
        *(const __attribute__((address_space(3))) bf16x8*)(ep + row * C::WN + ((j ^ sw) << 3));
    if (n < cols_valid && wm0 + row < u.rows_valid)
      *(u32x4*)(a.Y + (size_t)(u.r0 + wm0 + row) * a.ypitch + n0 + n) = __builtin_bit_cast(u32x4, v);
  }
}

// The up-projection's outputs: a lane holds the gate (accumulators 0..7) and
// the up (8..15) values of the same 8 outputs.
template <class C>
__device__ __forceinline__ void small_store(const G1Args& a, f32x16 (&acc)[C::NB][C::MB],
                                            uint16_t* smem, const SmallUnit& u, int wave, int lane,
                                            int wn0, int wm0, int n0, int cols_valid) {
  const int h = lane >> 5;
#pragma unroll
  for (int mb = 0; mb < C::MB; ++mb) {
    const int row = wm0 + 32 * mb + (lane & 31);
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb) {
      bf16x8 v;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float g = acc[nb][mb][i];
        const float w = acc[nb][mb][8 + i];
        v[i] = (__bf16)(g / (1.f + __expf(-g)) * w);
      }
      if (wn0 + 32 * nb < cols_valid && row < u.rows_valid)
        *(u32x4*)(a.xout + (size_t)(u.r0 + row) * a.I + (n0 + wn0) / 2 + 16 * nb + 8 * h) =
            __builtin_bit_cast(u32x4, v);
    }
  }
}

// A workgroup's share of the token -> rows inverse map, built beside its
// unit: the token ids load with the expert offsets, the counters' atomics go
// out before the operand loads, and their results are used after the unit.
template <int kThr>
struct RowShare {
  u64 epoch = 0, cnt_epoch = 0;
  RowPlace mine;
  int per = 0, row = -1, tok = -1;

  __device__ __forceinline__ void load(const KArgs& a) {
    epoch = launch_epoch(a);
    cnt_epoch = (epoch & ((1ull << (64 - kCntBits)) - 1)) << kCntBits;
    per = (int)((a.rows + gridDim.x - 1) / gridDim.x);
    const long long r = (long long)blockIdx.x * per + threadIdx.x;
    if ((int)threadIdx.x < per && r < a.rows) {
      row = (int)r;
      tok = a.token_ids[r];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0)
      __hip_atomic_store(a.map_epoch, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ __forceinline__ bool valid(const KArgs& a, int t) {
    if (t >= 0 && t < a.T) return true;
    __hip_atomic_fetch_or(a.status, kStBadRouting, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
  }
  __device__ __forceinline__ void claim(const KArgs& a, int rows_dev) {
    if (row >= rows_dev) row = -1;
    if (row >= 0 && !valid(a, tok)) row = -1;
    // more rows than threads in the share: the rest at once
    for (int i = threadIdx.x + kThr; i < per; i += kThr) {
      const long long r = (long long)blockIdx.x * per + i;
      if (r >= rows_dev) break;
      const int t = a.token_ids[r];
      if (!valid(a, t)) continue;
      RowPlace p;
      p.take(a, t, cnt_epoch);
      p.place(a, (int)r, t, cnt_epoch);
    }
    if (row >= 0) mine.take(a, tok, cnt_epoch);
  }
  __device__ __forceinline__ void finish(const KArgs& a) {
    if (row >= 0) mine.place(a, row, tok, cnt_epoch);
  }
  // the up-projection needs no inverse map
  __device__ __forceinline__ void load(const G1Args&) {}
  __device__ __forceinline__ void claim(const G1Args&, int) {}
  __device__ __forceinline__ void finish(const G1Args&) {}
};

// The unit's tile, by C::kThr threads with the ring at smem; `meanwhile` runs
// while the ring fills.
struct Nothing {
  __device__ __forceinline__ void operator()() const {}
};
template <class C, class Args, class Meanwhile = Nothing>
__device__ __forceinline__ void small_tile(const Args& a, uint16_t* smem, const SmallUnit& u,
                                           Meanwhile meanwhile = Meanwhile()) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n0 = u.n0, N = small_n(a);
  const int cols_valid = min(C::BN, N - n0);
  SmallCtx<C> t;
  t.lds = lds_addr(smem);
  const int ldb = gemm_ldb(a);
  t.rb = buffer_rsrc(gemm_b(a, u.e) + n0, ((long long)gemm_k(a) * ldb - n0) * 2);
  t.ra = buffer_rsrc(gemm_a_base(a, u.r0), gemm_a_bytes(a, u.r0));
#pragma unroll
  for (int q = 0; q < C::WL; ++q) {
    const int i = C::WL * wave + q;
    const int flat = 64 * i + lane;   // 16-byte chunk of the stage
    const int krow = flat / C::WC;
    const int wc = (flat % C::WC) ^ C::wswz(krow);
    t.wk[q] = krow;
    t.wo[q] = 8 * wc < cols_valid ? 16u * (uint32_t)wc + 2u * (uint32_t)krow * (uint32_t)ldb
                                  : kOutOfRange;
  }
#pragma unroll
  for (int q = 0; q < C::XL; ++q) {
    const int row = 64 / C::XC * (C::XL * wave + q) + lane / C::XC;
    const int lc = (lane % C::XC) ^ ((row / C::kXPerLine) % C::XC);
    t.xk[q] = 8 * lc;
    t.xo[q] = row < u.rows_valid ? small_a_off(a, u.r0, row) + 16u * (uint32_t)lc : kOutOfRange;
  }
  const int wn0 = (wave % C::WNW) * C::WN;
  const int wm0 = (wave / C::WNW) * C::WM;
  int offA[C::NB];
  {
    const int j = lane & 15;
    const int krow = 8 * (lane >> 5) + (j >> 2);
    const int uu = j & 3;
    const int rg = (lane >> 4) & 1;
#pragma unroll
    for (int nb = 0; nb < C::NB; ++nb) {
      const int col = wn0 + 32 * nb + 16 * rg + 8 * (uu & 1) + 4 * (uu >> 1);
      offA[nb] = C::kXElems + krow * C::BN + (((col >> 3) ^ C::wswz(krow)) << 3) + (col & 7);
    }
  }
  int offB[C::KS];
  {
    const int m = wm0 + (lane & 31);
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
      const int c = 2 * ks + (lane >> 5);
      offB[ks] = m * C::BK + ((c ^ ((m / C::kXPerLine) % C::XC)) << 3);
    }
  }
  const int nk = (gemm_k(a) + C::BK - 1) / C::BK;
#pragma unroll
  for (int s = 0; s + 1 < C::S; ++s) small_issue<C>(a, t, s, s, wave);
  meanwhile();
  f32x16 acc[C::NB][C::MB];
#pragma unroll
  for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
    for (int mb = 0; mb < C::MB; ++mb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[nb][mb][i] = 0.f;
  int slot = 0, fill = C::S - 1;
  for (int kt = 0; kt < nk; ++kt) {
    waitcnt_vm<(C::S - 2) * C::LPS>();
    block_barrier();
    small_issue<C>(a, t, kt + C::S - 1, fill, wave);
    lds_u16* st = (lds_u16*)(uintptr_t)(t.lds + (uint32_t)slot * (C::kSlot * 2));
    auto frags = [&](int ks, bf16x8 (&af)[C::NB], bf16x8 (&bm)[C::MB]) {
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb) {
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_i16x4*)(st + offA[nb] + ks * 16 * C::BN));
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_i16x4*)(st + offA[nb] + ks * 16 * C::BN + 4 * C::BN));
        const i16x8 w = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        af[nb] = __builtin_bit_cast(bf16x8, w);
      }
#pragma unroll
      for (int mb = 0; mb < C::MB; ++mb)
        bm[mb] = *(const __attribute__((address_space(3))) bf16x8*)(st + offB[ks] + mb * 32 * C::BK);
    };
    auto mfmas = [&](const bf16x8 (&af)[C::NB], const bf16x8 (&bm)[C::MB]) {
#pragma unroll
      for (int nb = 0; nb < C::NB; ++nb)
#pragma unroll
        for (int mb = 0; mb < C::MB; ++mb)
          acc[nb][mb] =
              __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[nb], bm[mb], acc[nb][mb], 0, 0, 0);
    };
    // the next step's fragments are read ahead of this step's MFMAs
    bf16x8 af[2][C::NB], bm[2][C::MB];
    frags(0, af[0], bm[0]);
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
      if (ks + 1 < C::KS) frags(ks + 1, af[(ks + 1) & 1], bm[(ks + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(af[ks & 1], bm[ks & 1]);
    }
    slot = slot + 1 == C::S ? 0 : slot + 1;
    fill = fill + 1 == C::S ? 0 : fill + 1;
  }
  waitcnt_vm<0>();   // no load may land in the ring under the epilogue
  block_barrier();
  small_store<C>(a, acc, smem, u, wave, lane, wn0, wm0, n0, cols_valid);
}

// Where the last column block has at most 128 columns, tiles 256 wide leave
// it to 128 x 128 ones (mixed_edge), with as many threads and no more LDS.
using SmallTile128 = SmallTile<128, 128, 8, 4, 2>;   // 64 KB of LDS, two per CU
constexpr int kEdge = kBN / 2;
__host__ __device__ inline bool mixed_edge(int N) { return N % kBN != 0 && N % kBN <= kEdge; }

template <class C, class Args>
__global__ void __launch_bounds__(C::kThr) small_gemm_kernel(Args a) {
  __shared__ __attribute__((aligned(1024))) uint16_t smem[C::S * C::kSlot];
  RowShare<C::kThr> share;
  share.load(a);
  int rows_dev;
  const SmallUnit u = small_unit<C::BM, C::BN>(a.offsets, a.rows, a.E,
                                               (small_n(a) + C::BN - 1) / C::BN, a.status, &rows_dev);
  share.claim(a, rows_dev);
  if (u.ok) {
    if constexpr (C::BN == kBN) {
      static_assert(C::BM == SmallTile128::BM && C::kThr == SmallTile128::kThr &&
                        C::S * C::kSlot >= SmallTile128::S * SmallTile128::kSlot,
                    "the edge tile in the wide tile's place");
      if (mixed_edge(small_n(a)) && u.n0 + kEdge >= small_n(a))
        small_tile<SmallTile128>(a, smem, u);
      else
        small_tile<C>(a, smem, u);
    } else {
      small_tile<C>(a, smem, u);
    }
  }
  share.finish(a);
}

// ---- large batches: full 256 x 256 tiles, the rest in smaller ones -----------------
// P workgroups (one per CU) run the tiles with 256 rows, chained as in the
// persistent kernel, and after them the smaller tiles, which fill the partial
// last round and keep the padding small:
//  * 256 x 128 tiles over the right edge, where the last column block has at
//    most 128 columns (2 I = 1408 is five blocks and a half);
//  * 128 x 256 tiles over the rows past each expert's last full tile.
// The stage starts further workgroups for those, 2 P at most, as the CUs become
// free.  The up-projection gives each of its P workgroups as many, after its full
// tiles, as the plan says for one with and one without a tile of the last round.
// (With a workgroup for every smaller tile that the host's bound allows, most
// found out for themselves, on a CU of their own, that there was nothing for
// them: up-projection, H = 2048, I = 704, E = 32, T = 16384 531.8 us, now 520.7;
// H = 512, I = 128, E = 1024, 100 rows each 135, now 86.  The stage's P workgroups
// wait for a full tile's stores before the first smaller one: 388.4 us against
// 383.3 with further ones, which start meanwhile.  Handed out by counters in the
// workspace, the smaller tiles waited for the counters: H = 2048, I = 512, E =
// 256, top-8, T = 8192, Zipf 1.0, 306 us, by index 280.)
using MixedEdge = SmallTile<256, 128, 8, 2, 3>;
using MixedBottom = SmallTile<128, 256, 8, 4, 3>;
static_assert(sizeof(Smem) >= MixedEdge::S * MixedEdge::kSlot * 2 &&
                  sizeof(Smem) >= MixedBottom::S * MixedBottom::kSlot * 2,
              "the smaller tiles' rings overlay the whole of Smem");

// How a launch's rows and columns are cut: an expert has (count + pad) / 256
// full m-tiles, the rows left are bottoms; `edge`: the last column block is
// left to the edge tiles, else it is an ordinary (partly empty) block.
struct MixedPlan {
  int pad;
  bool edge;
  int blocks;                // column blocks of the full tiles and the bottoms
  int full, edges, bottoms;  // full tiles, edge tiles, bottom m-units
  int early, late;           // smaller tiles of a workgroup without / with a last full tile
};

__device__ __forceinline__ int mixed_bottoms(int count, int pad) {
  return (max(0, count - (count + pad) / kBM * kBM) + MixedBottom::BM - 1) / MixedBottom::BM;
}

// x / n for 0 <= x < 2^24 and n > 0, by one reciprocal.
__device__ __forceinline__ int small_div(int x, int n) {
  int q = (int)((float)x * __builtin_amdgcn_rcpf((float)n));
  q -= q * n > x;
  q += (q + 1) * n <= x;
  return q;
}

// The time of `full` tiles of fc each on P workgroups followed by `small`
// tiles of hc each, early on a workgroup without a last full tile and late on
// one with it: as few as hold them all.
__device__ __forceinline__ float mixed_time(int full, int small, int P, int fc, int hc, int& early,
                                            int& late) {
  const int rounds = small_div(full, P), rem = full - rounds * P;
  int t = rem > 0 ? fc : 0;
  early = late = 0;
  if (small > 0) {
    const int behind = small_div(fc - 1, hc) + 1;   // small tiles a full one takes the place of
    for (early = small_div(small, P);; ++early) {   // small / P at least
      late = max(0, early - behind);
      if ((P - rem) * early + rem * late >= small) {
        t = max(t, early * hc);
        break;
      }
      const int t_late = fc + (late + 1) * hc;
      if (t_late < (early + 1) * hc && (P - rem) * early + rem * (late + 1) >= small) {
        ++late;
        t = max(t, t_late);
        break;
      }
    }
  }
  return (float)rounds * fc + t;
}

// The plan with the least time, from the expert counts alone, so every wave
// of the launch finds the same one.  Tile times for nk 64-deep stages, in
// 10 ns, measured: 704 and 2048 deep, a full tile 1.5 us a stage + 4 us, a
// smaller one 0.93 us a stage + 5.5 us, as it starts on its own.  An expert of
// one m-tile streams its weights from HBM for it alone: the stage (256 to 1536
// deep, E = 512 and 1024) 1.66 us a stage + 1.5 us for a full tile and 1.28 us +
// 4.5 us for a smaller one, the up-projection (512 to 4096 deep) 1.66 us + 5.5 us
// and 1.36 us + 4.2 us.  So the stage's full tiles stay whole for such
// experts below 8 stages: H = 2048, I = 256, E = 1024, 16 rows each, 284 us
// against 328; I = 768 takes 640 with the smaller ones against 698.
template <class Args>
__device__ __forceinline__ MixedPlan mixed_plan(const Args& a, int P) {
  const int lane = threadIdx.x & 63;
  const int N = small_n(a), nk = min(1024, (gemm_k(a) + kBK - 1) / kBK);
  // m-tiles; experts with 1..128, 129..192 rows past them, and those of one m-tile
  int all = 0, low = 0, mid = 0, one = 0, one_low = 0, one_mid = 0;
  auto count_tiles = [&](auto k) {
    constexpr int K = decltype(k)::value;
    for (int e0 = 0; e0 < a.E; e0 += 64 * K) {
      const ExpertRows<K> r(a.offsets, a.rows, a.E, e0);
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int past = r.count[i] % kBM;
        const u64 is_low = __ballot(past >= 1 && past <= 128), is_mid = __ballot(past >= 129 && past <= 192);
        const u64 is_one = __ballot(r.count[i] >= 1 && r.count[i] <= kBM);
        low += __builtin_popcountll(is_low);
        mid += __builtin_popcountll(is_mid);
        one += __builtin_popcountll(is_one);
        one_low += __builtin_popcountll(is_low & is_one);
        one_mid += __builtin_popcountll(is_mid & is_one);
      }
      all += r.sum([](int count) { return (count + kBM - 1) / kBM; });
    }
  };
  if (a.E <= 64)
    count_tiles(std::integral_constant<int, 1>());
  else
    count_tiles(std::integral_constant<int, 4>());
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) all += __shfl_xor(all, d);
  all = __builtin_amdgcn_readfirstlane(all);
  // Offsets that decrease (they are flagged) can give every expert all rows.  The
  // stage then has no tiles, as in the persistent kernel (the up-projection, as
  // before, computes them, E times the rows at most).
  if (!RowGather<Args>::on && all > (int)((a.rows + kBM - 1) / kBM) + a.E)
    return {kBM - 1, false, 0, 0, 0, 0, 0, 0};
  // one round of full tiles holds everything: nothing to weigh
  const int whole = (N + kBN - 1) / kBN;
  if (all <= small_div(P, whole)) return {kBM - 1, false, whole, all * whole, 0, 0, 0, 0};
  const int fc_far = RowGather<Args>::on ? 166 * nk + 550 : 166 * nk + 150;
  const int hc_far = RowGather<Args>::on ? 136 * nk + 420 : 128 * nk + 450;
  // lane l weighs plan l: up to 192, 128 or no rows (l % 3) past an expert's
  // last full tile, with the edge tiles from l = 3 on
  const int p = lane % 3;
  const bool edge = lane >= 3;
  const int blocks = edge ? N / kBN : (N + kBN - 1) / kBN;
  const int m_full = all - (p == 0 ? low + mid : p == 1 ? low : 0);
  const int full = m_full * blocks;
  const int bottoms = p == 0 ? low + 2 * mid : p == 1 ? low : 0;
  const int edges = edge ? all : 0;
  float cost = 3e38f;
  int early = 0, late = 0;
  const long long small_all = edges + (long long)bottoms * blocks;
  // (past 2^22 tiles, where small_div ends, only plan 2: full tiles alone)
  if (lane < (mixed_edge(N) ? 6 : 3) && full < (1 << 22) && small_all < (1 << 22)) {
    const int small = (int)small_all;
    // mean times, by the share of the tiles whose experts have no other
    const int one_full = one - (p == 0 ? one_low + one_mid : p == 1 ? one_low : 0);
    const int one_small = (p == 0 ? one_low + 2 * one_mid : p == 1 ? one_low : 0) * blocks;
    int fc = 150 * nk + 400, hc = 93 * nk + 550;
    if (m_full > 0) fc += (int)((fc_far - fc) * ((float)one_full / m_full));
    if (small > 0) hc += (int)((hc_far - hc) * ((float)one_small / small));
    // the average load breaks ties (and counts for the power it takes); the
    // smaller tiles have to save a sixth of a full one (one round of full tiles
    // for everything 35.6 us, with smaller ones on its idle CUs 39.7)
    cost = mixed_time(full, small, P, fc, hc, early, late) +
           ((float)full * fc + (float)small * hc) * 0.25f / P + (small > 0 ? fc / 6 : 0);
  }
  int best = 2;
  float least = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cost), 2));
#pragma unroll
  for (int l = 0; l < 6; ++l) {
    const float c = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cost), l));
    if (c < least) {
      least = c;
      best = l;
    }
  }
  MixedPlan plan;
  plan.pad = best % 3 == 0 ? 63 : best % 3 == 1 ? 127 : kBM - 1;
  plan.edge = best >= 3;
  plan.blocks = __builtin_amdgcn_readlane(blocks, best);
  plan.full = __builtin_amdgcn_readlane(full, best);
  plan.edges = __builtin_amdgcn_readlane(edges, best);
  plan.bottoms = __builtin_amdgcn_readlane(bottoms, best);
  plan.early = __builtin_amdgcn_readlane(early, best);
  plan.late = __builtin_amdgcn_readlane(late, best);
  return plan;
}

// The stage's first workgroup leaves the plan in the workspace, tagged with the
// launch, for those behind the first P, which start later: one that finds it
// needs no plan of its own, one that does not (nothing waits) makes it.  (Two
// rounds of idle workgroups with plans of their own, H = 512, I = 128, E = 1024,
// 16 rows each: 67 us, now 59.)
__device__ __forceinline__ void leave_plan(const KArgs& a, const MixedPlan& plan, u64 epoch) {
  const u64 tag = (u64)(uint32_t)epoch << 32;   // (its low half is never 0)
  const uint32_t w[3] = {(uint32_t)plan.pad << 1 | plan.edge, (uint32_t)plan.edges, (uint32_t)plan.bottoms};
#pragma unroll
  for (int i = 0; i < 3; ++i)
    __hip_atomic_store(a.plan_left + i, tag | w[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ MixedPlan find_plan(const KArgs& a, int P) {
  const uint32_t tag = (uint32_t)launch_epoch(a);
  u64 w[3];
  bool all = true;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    w[i] = __hip_atomic_load(a.plan_left + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    all &= (uint32_t)(w[i] >> 32) == tag;
  }
  if (!__all(all)) return mixed_plan(a, P);
  MixedPlan plan = {};
  const int first = __builtin_amdgcn_readfirstlane((int)(uint32_t)w[0]);
  plan.pad = first >> 1;
  plan.edge = first & 1;
  plan.blocks = plan.edge ? a.H / kBN : (a.H + kBN - 1) / kBN;
  plan.edges = __builtin_amdgcn_readfirstlane((int)(uint32_t)w[1]);
  plan.bottoms = __builtin_amdgcn_readfirstlane((int)(uint32_t)w[2]);
  return plan;   // (full, early and late are the first P's)
}

// A workgroup's smaller tiles: first, first + step, ... below end, `count` at
// most.
struct MixedShare {
  int first, step, count, end;
  __device__ __forceinline__ int next() {   // -1 at the end
    const int j = first;
    first += step;
    return count-- > 0 && j < end ? j : -1;
  }
};
// Those of the up-projection's workgroup b of P, the first full % P of which
// have a tile of the last round.  Each XCD (b mod 8) has a range of neighbouring
// units, as long as its workgroups' share of the whole; those without a last
// full tile take its front in turns, the others its back.
__device__ __forceinline__ MixedShare mixed_share(const MixedPlan& plan, int b, int P) {
  const int rem = plan.full % P;
  const int units = plan.edges + plan.bottoms * plan.blocks;
  auto on_xcd = [](int n, int x) { return (n + 7 - x) >> 3; };   // workgroups below n on XCD x
  int before = 0, all = 0, mine = 0;   // how many the workgroups of XCDs hold
  for (int x = 0; x < 8; ++x) {
    const int with = on_xcd(rem, x), cap = (on_xcd(P, x) - with) * plan.early + with * plan.late;
    if (x < (b & 7)) before += cap;
    if (x == (b & 7)) mine = cap;
    all += cap;
  }
  const int lo = (int)((long long)units * before / all);
  const int with = on_xcd(rem, b & 7), without = on_xcd(P, b & 7) - with;
  MixedShare sh;
  sh.end = (int)((long long)units * (before + mine) / all);
  if (b < rem)
    sh.first = lo + without * plan.early + (b >> 3), sh.step = with, sh.count = plan.late;
  else
    sh.first = lo + (b >> 3) - with, sh.step = without, sh.count = plan.early;
  return sh;
}

// The smaller tiles that the stage's i-th workgroup behind the first P takes: of
// its XCD's (i mod 8) eighth of the units those of its index, one in each round
// of the `per` workgroups there.
__device__ __forceinline__ MixedShare mixed_behind(const KArgs& a, const MixedPlan& plan, int i) {
  const int all = plan.edges + plan.bottoms * plan.blocks, chunk = (all + 7) >> 3;
  const int lo = (i & 7) * chunk;
  const int per = ((int)gridDim.x - a.P) >> 3;   // (a multiple of eight workgroups)
  return {lo + (i >> 3), per, chunk, min(lo + chunk, all)};
}

// Unit `i` of the smaller tiles: edges first, then bottoms; by each wave for
// itself.
template <int K, class Args>
__device__ __forceinline__ SmallUnit mixed_unit_of(const Args& a, const MixedPlan& plan, int i, bool edge) {
  SmallUnit u = {0, 0, 0, 0, true};
  const int per = edge ? 1 : plan.blocks;   // column blocks per m-unit
  const int unit = edge ? i : i - plan.edges;
  const int mt = unit / per;
  auto units = [=](int count) { return edge ? (count + kBM - 1) / kBM : mixed_bottoms(count, plan.pad); };
  for (int carry = 0, e0 = 0; e0 < a.E; e0 += 64 * K) {
    const ExpertRows<K> r(a.offsets, a.rows, a.E, e0);
    const int v = wave_prefix(r.sum(units));
    const int sum = __builtin_amdgcn_readlane(v, 63);
    if (mt >= carry + sum) {
      carry += sum;
      continue;
    }
    const ExpertUnit x = find_expert(r, e0, mt, units, carry, v);
    const int within = unit - x.first * per;
    const int nt = within / x.n, mi = within - nt * x.n;
    const int row = edge ? mi * kBM : (x.count + plan.pad) / kBM * kBM + mi * MixedBottom::BM;
    u.e = x.e;
    u.r0 = x.start + row;
    u.rows_valid = min(edge ? kBM : MixedBottom::BM, x.count - row);
    u.n0 = edge ? plan.blocks * kBN : nt * kBN;
    return u;
  }
  u.ok = false;   // (never: i is below the plan's units)
  return u;
}
// (a negative i: none)
template <class Args>
__device__ __forceinline__ SmallUnit mixed_unit(const Args& a, const MixedPlan& plan, int i) {
  if (i < 0) return {0, 0, 0, 0, false};
  const bool edge = i < plan.edges;
  return a.E <= 64 ? mixed_unit_of<1>(a, plan, i, edge) : mixed_unit_of<4>(a, plan, i, edge);
}

__device__ __forceinline__ void mixed_prologue(Smem& sm, const KArgs& a, const MixedPlan& plan) {
  if (threadIdx.x == 0) {
    sm.epoch = launch_epoch(a);   // load_experts synchronises
    if (blockIdx.x == 0) {
      __hip_atomic_store(a.map_epoch, sm.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      leave_plan(a, plan, sm.epoch);
    }
  }
}
__device__ __forceinline__ void mixed_prologue(Smem&, const G1Args&, const MixedPlan&) {}
__device__ __forceinline__ void mixed_inverse_map(const Smem& sm, const KArgs& a) {
  consumer_prologue(sm, a, (long long)sm.start[a.E - 1] + sm.count[a.E - 1], false, a.P, false);
  waitcnt_vm<0>();   // nothing the compiler tracks stays in flight in the tile loop
}
__device__ __forceinline__ void mixed_inverse_map(const Smem&, const G1Args&) {}

// The smaller tiles of a workgroup's share, the ring over sm.  The next one is
// looked up while a tile fills its ring: after its epilogue the offsets' loads
// would wait for its stores.  (Every wave of the workgroup is past its use of sm
// on entry; the barrier keeps a tile's loads behind the one before.)
template <class Args>
__device__ __forceinline__ void mixed_small_tiles(Smem& sm, const Args& a, const MixedPlan& plan,
                                                  MixedShare share) {
  uint16_t* ring = reinterpret_cast<uint16_t*>(&sm);
  int j = share.next();
  SmallUnit u = mixed_unit(a, plan, j);
  while (u.ok) {
    const bool edge = j < plan.edges;
    SmallUnit u_next;
    auto look_up = [&] {
      j = share.next();
      u_next = mixed_unit(a, plan, j);
    };
    if (edge)
      small_tile<MixedEdge>(a, ring, u, look_up);
    else
      small_tile<MixedBottom>(a, ring, u, look_up);
    block_barrier();
    u = u_next;
  }
}

template <class Args>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
mixed_gemm_kernel(Args a) {
  constexpr bool kUp = RowGather<Args>::on;   // the up-projection
  __shared__ __attribute__((aligned(1024))) Smem sm;
  const int P = a.P;
  if constexpr (!kUp) {
    if ((int)blockIdx.x >= P) {
      const MixedPlan plan = find_plan(a, P);
      mixed_small_tiles(sm, a, plan, mixed_behind(a, plan, (int)blockIdx.x - P));
      return;
    }
  }
  const MixedPlan plan = mixed_plan(a, P);
  // (what the smaller tiles need later waits in LDS, in the token bands' room)
  MixedPlan& kept_plan = *reinterpret_cast<MixedPlan*>(sm.band_pre);
  MixedShare& kept_share = *reinterpret_cast<MixedShare*>(sm.band_pre + 16);
  static_assert(sizeof(MixedPlan) <= 64 && sizeof(sm.band_pre) >= 64 + sizeof(MixedShare), "room");
  if (kUp && threadIdx.x == 0) {   // load_experts synchronises
    kept_plan = plan;
    if (plan.early + plan.late > 0)
      kept_share = mixed_share(plan, (int)blockIdx.x, P);
    else
      kept_share = {0, 0, 0, 0};
  }
  mixed_prologue(sm, a, plan);
  load_experts(sm, a, plan.pad);
  a.ntps = plan.blocks;   // for decode_tile
  const int total = sm.tile_prefix[a.E] * a.ntps;
  const int full = total / P * P;   // whole rounds; the rest one each, spread over the XCDs
  auto tile_of = [&](int k) {
    if (k * P < full) return k * P + compute_index((int)blockIdx.x, 0, P);
    if (k * P == full && (int)blockIdx.x < total - full)
      return full + compute_index((int)blockIdx.x, 0, total - full);
    return -1;
  };
  const int nk = (gemm_k(a) + kBK - 1) / kBK;
  TileInfo cur = {0, 0, 0, 0, 0, 0};
  TileCtx tctx;
  bool filled = false;
  int g = tile_of(0);
  if (g >= 0) {
    cur = decode_tile(sm, a, total, g);
    if constexpr (!kUp) {   // its loads fly during the inverse map's atomics
      const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
      tctx = make_ctx(sm, a, cur, wave);
      issue_prologue(a, tctx, nk, 0, wave);
      filled = true;
    }
  }
  mixed_inverse_map(sm, a);
  int base = 0;
  for (int k = 0; g >= 0; ++k) {
    const int g_next = tile_of(k + 1);
    const bool next = g_next >= 0;
    const TileInfo nt = next ? decode_tile(sm, a, total, g_next) : cur;
    u64 t_mid[2];
    compute_tile(sm, a, cur, filled, next, nt, base, t_mid, tctx);
    base = (base + nk) % kStages;
    filled = next;
    cur = nt;
    g = g_next;
  }
  if constexpr (kUp) {
    const MixedPlan rest = kept_plan;
    const MixedShare share = kept_share;
    waitcnt_vm<63>();   // (these reads; its own loads compute_tile has waited for)
    block_barrier();
    mixed_small_tiles(sm, a, rest, share);
  }
}

// out[t, :] for every token: one wave per token and 256 columns.  The
// token's count, its rows (in inverse-map order, sorted by rank across the
// lanes) and then its gates and Y rows are two dependent round trips (3.0 us
// for one token); with many tokens it is bound by the Y rows read and the
// output written (T = 16384, H = 2048, top-6: 537 MB in 85.5 us, 6.3 TB/s).
// Only the rows a token has are read: padding its list to eight with repeated
// rows cost 8% of the stage at top-4, T = 16384.  The first launch built the
// inverse map under launch epoch *map_epoch; storing that as the workspace's
// completed epoch ends the launch pair (only the first launch reads it).
constexpr int kSmallCombineWaves = 4;

// Adds acc, this lane's columns 4 lane .. 4 lane + 3 of the 256 at o (of which
// `cols` exist), each atomic on 64 neighbouring columns (on every fourth column
// it touches four times the lines).
__device__ __forceinline__ void add_block(float* o, int cols, const float (&acc)[4]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = __builtin_amdgcn_ds_bpermute(4 * (16 * i + (lane >> 2)), __float_as_int(acc[e]));
    const int even = lane & 1 ? v[1] : v[0], odd = lane & 1 ? v[3] : v[2];
    const int c = 64 * i + lane;
    if (c < cols) atomic_add_f32(o + c, __int_as_float(lane & 2 ? odd : even));
  }
}

// Rows j0 .. j0+U-1 of a token (its sorted rows in lanes of rs, gates in gs)
// at CB column blocks: all loads first, then the sums in ascending order.
template <int U, int CB, bool kNtLoad>
__device__ __forceinline__ void small_gather(const uint16_t* y, int ypitch, int j0, int rs, int gs,
                                             const int (&col)[CB], float (&acc)[CB][4]) {
  u32x2 v[U][CB];
#pragma unroll
  for (int q = 0; q < U; ++q) {
    const uint16_t* yr = y + (size_t)__builtin_amdgcn_readlane(rs, j0 + q) * ypitch;
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const u32x2* p = (const u32x2*)(yr + col[b]);
      v[q][b] = kNtLoad ? __builtin_nontemporal_load(p) : *p;
    }
  }
#pragma unroll
  for (int q = 0; q < U; ++q) {
    const float g = __int_as_float(__builtin_amdgcn_readlane(gs, j0 + q));
#pragma unroll
    for (int b = 0; b < CB; ++b) fma4(acc[b], g, v[q][b]);
  }
}

template <int CB, bool kNtLoad, bool kScatter>
__device__ __forceinline__ void small_combine_unit(const KArgs& a, u64 epoch, long long unit,
                                                   int cbs) {
  const int lane = threadIdx.x & 63;
  const int t = (int)(unit / cbs);
  const int c0 = (int)(unit - (long long)t * cbs) * 256 * CB + 4 * lane;
  int col[CB];
#pragma unroll
  for (int b = 0; b < CB; ++b) col[b] = c0 + 256 * b < a.H ? c0 + 256 * b : 0;
  const u64 cnt_epoch = (epoch & ((1ull << (64 - kCntBits)) - 1)) << kCntBits;
  const int K = a.topk;
  const uint32_t have = epoch_count(a.tok_cnt[t], cnt_epoch);
  int r = lane < K ? a.inv[(long long)t * K + lane] : 0;
  const int n = __builtin_amdgcn_readfirstlane((int)(have < (uint32_t)K ? have : (uint32_t)K));
  float g = 0.f;
  if (lane < n) g = a.gate_w[r];
  // ascending row order: lane q < n sends its row to the lane of its rank
  int rank = lane;
  if (lane < n) rank = 0;
  for (int q = 0; q < n; ++q) {
    const int rq = __builtin_amdgcn_readlane(r, q);
    if (lane < n) rank += rq < r;
  }
  const int rs = __builtin_amdgcn_ds_permute(4 * rank, r);
  const int gs = __builtin_amdgcn_ds_permute(4 * rank, __float_as_int(g));
  float acc[CB][4];
#pragma unroll
  for (int b = 0; b < CB; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[b][i] = 0.f;
  int j = 0;
  for (; j + 8 <= n; j += 8) small_gather<8, CB, kNtLoad>(a.Y, a.ypitch, j, rs, gs, col, acc);
  if (n - j >= 6) small_gather<6, CB, kNtLoad>(a.Y, a.ypitch, j, rs, gs, col, acc), j += 6;
  if (n - j >= 4) small_gather<4, CB, kNtLoad>(a.Y, a.ypitch, j, rs, gs, col, acc), j += 4;
  if (n - j >= 2) small_gather<2, CB, kNtLoad>(a.Y, a.ypitch, j, rs, gs, col, acc), j += 2;
  if (n - j >= 1) small_gather<1, CB, kNtLoad>(a.Y, a.ypitch, j, rs, gs, col, acc);
  // (mode 1, a token with more than topk rows: the first launch zeroed its
  // output, and small_add_listed adds the others)
  const bool add = kScatter && __builtin_amdgcn_readfirstlane(have) > (uint32_t)K;
#pragma unroll
  for (int b = 0; b < CB; ++b) {
    float* o = a.out + (size_t)t * a.H + c0 + 256 * b;
    if (add)
      add_block(o - 4 * lane, a.H - (c0 - 4 * lane + 256 * b), acc[b]);
    else if (c0 + 256 * b < a.H)
      __builtin_nontemporal_store(f32x4{acc[b][0], acc[b][1], acc[b][2], acc[b][3]}, (f32x4*)o);
  }
}

// Mode 1: the `listed` rows past their token's topk, eight at a time, spread over
// every wave of the launch; neighbours of one token are summed before they are
// added.  (One wave per token and column block for its part of the list, a load
// at a time, took 13.2 ms where half of T = 8192, top-8, H = 1024 rows are one
// token's; now 0.23.)
template <int CB, bool kNtLoad>
__device__ __forceinline__ void small_add_listed(const KArgs& a, int listed, int cbs) {
  constexpr int U = 8;
  const int lane = threadIdx.x & 63;
  const int32_t* list = a.inv + (size_t)a.T * a.topk;
  const long long groups = (listed + U - 1) / U;
  for (long long k = (long long)blockIdx.x * kSmallCombineWaves +
                     __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
       k < groups * cbs; k += (long long)gridDim.x * kSmallCombineWaves) {
    const long long group = k / cbs;
    const int c0 = (int)(k - group * cbs) * 256 * CB + 4 * lane;
    const int n = min(U, (int)(listed - group * U));
    const int r = list[group * U + min(lane, n - 1)];
    const int t = a.token_ids[r], g = __float_as_int(a.gate_w[r]);
    u32x2 v[U][CB];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const uint16_t* yr = a.Y + (size_t)__builtin_amdgcn_readlane(r, q) * a.ypitch;
#pragma unroll
      for (int b = 0; b < CB; ++b) {
        const u32x2* p = (const u32x2*)(yr + (c0 + 256 * b < a.H ? c0 + 256 * b : 0));
        v[q][b] = kNtLoad ? __builtin_nontemporal_load(p) : *p;
      }
    }
    float acc[CB][4] = {};
#pragma unroll
    for (int q = 0; q < U; ++q) {
      if (q >= n) break;
      const int tq = __builtin_amdgcn_readlane(t, q);
#pragma unroll
      for (int b = 0; b < CB; ++b) fma4(acc[b], __int_as_float(__builtin_amdgcn_readlane(g, q)), v[q][b]);
      if (q + 1 < n && __builtin_amdgcn_readlane(t, q + 1 < U ? q + 1 : q) == tq) continue;
#pragma unroll
      for (int b = 0; b < CB; ++b) {
        const int cb = c0 - 4 * lane + 256 * b;
        add_block(a.out + (size_t)tq * a.H + cb, a.H - cb, acc[b]);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[b][i] = 0.f;
      }
    }
  }
}

// kScatter: mode 1
template <int CB, bool kNtLoad, bool kScatter>
__global__ void __launch_bounds__(kSmallCombineWaves * 64) small_combine_kernel(KArgs a) {
  const u64 epoch =
      __hip_atomic_load(a.map_epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const u64 over = kScatter ? __hip_atomic_load(a.over_cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  if (blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(a.epoch_word, (uint32_t)(epoch + 1) == 0 ? epoch + 1 : epoch,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int cbs = (a.H + 256 * CB - 1) / (256 * CB);
  const long long units = (long long)a.T * cbs;
  for (long long unit = (long long)blockIdx.x * kSmallCombineWaves +
                        __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
       unit < units; unit += (long long)gridDim.x * kSmallCombineWaves)
    small_combine_unit<CB, kNtLoad, kScatter>(a, epoch, unit, cbs);
  if constexpr (kScatter) {
    const u64 cnt_epoch = (epoch & ((1ull << (64 - kCntBits)) - 1)) << kCntBits;
    const long long slots = (long long)a.T * a.topk, n = epoch_count(over, cnt_epoch);
    const int listed = __builtin_amdgcn_readfirstlane((int)(n < slots ? n : slots));
    if (listed > 0) small_add_listed<CB, kNtLoad>(a, listed, cbs);
  }
}
