// Large-M GEMM of the encoder layers (paper §III-B: the QKV, output
// projection and MLP products, eqs. 4-5), for calls whose row count M is known
// on the host: full encodes, top-k steps and the all-rows MLP.  The small-M
// kernel (gemm.hpp) streams the weights once and re-reads the A rows per 16-64
// columns; here each workgroup stages a tile of A rows and of W columns
// through LDS once per K chunk and all its waves multiply from there.
//
//   * output tile BM x BN per workgroup, 8 waves in a WR x WC grid, each wave
//     owning (BM / WR) x (BN / WC) outputs as 16x16 MFMA accumulators
//     (v_mfma_f32_16x16x32_bf16, fp32 accumulation).  The W fragment is the
//     first operand, so a lane ends up with 4 consecutive columns of one row:
//     the epilogue needs no exchange between lanes and its stores to the
//     operand-order buffers cover whole 512-byte runs;
//   * the K loop runs over slots of KD 32-deep chunks.  A chunk's operands are
//     BM / 16 A fragments and BN / 16 W fragments, each a contiguous kilobyte
//     in HBM (the compact rows and the packed weights are stored in MFMA
//     operand order), so one wave instruction (buffer_load_dwordx4 ... lds: 16
//     bytes per lane straight into LDS, no registers) stages one fragment.  A
//     ring of NS slots keeps NS - 2 or more in flight;
//   * the fragments of a step are read from LDS while the step before it is
//     multiplied, spread between its products together with the staging of a
//     slot further on; one barrier per slot.  The loop has no branch and no
//     wait that depends on the position: with the staging's bookkeeping in
//     branches a slot took 600-1000 clocks of it alone;
//   * a workgroup runs over several tiles (at most one workgroup per CU's
//     place is launched) and the ring runs on across them: the next tile's
//     first slots land while this tile's epilogue stores;
//   * the folded LayerNorm (QKV, MLP up) takes its row statistics on the
//     matrix cores from the staged A fragments (x * ones and the diagonal of
//     x * x^T), each wave for its share of the row tiles;
//   * each XCD takes a compact block of about sqrt(tiles / 8) row tiles by as
//     many column tiles, so its workgroups share their A and W tiles in its
//     L2 (the hardware deals workgroups to the XCDs round robin);
//   * partial sums (the MLP down projection while its tiles are fewer than
//     the CUs) may split K: split z takes a contiguous range of chunks and
//     writes its fp32 partial sums, which the row kernel adds in split order.
//
// Measured (MI355X; us per launch and TFLOP/s, weights from HBM): MLP down of
// 8192 rows (ViT-L) 75 -> 63 us, 1090; MLP up 106 -> 77, 890; QKV 79 -> 71, 725;
// MLP up of 1024 rows (So400m) 28 -> 22, QKV 20.7 -> 16, of 256 rows 14 -> 9.9.
// This staging alone runs at 41 B/clk per CU from a warm L2 (a bare loop of LDS
// DMA takes in 53, one of register loads 51: it is what the L2 delivers) and LDS
// reads alone at 240 B/clk; their sum is what bounds a 128 x 128 tile (no
// products: 72 of its 75 us).
//
// bf16 models only (fp32 models use the small-M kernel).  Results do not
// depend on the tile shape beyond the fp32 order of the MFMA accumulation,
// which is fixed (k ascending); no atomics.
#pragma once
#include "gemm.hpp"

namespace incvit {

constexpr int kTiledWaves = 8;

// LDS: the ring of NS slots, then (QKV, MLP up) the rows' sums and sums of
// squares [BM] float2
template <int BM, int BN, int KD, int NS>
__host__ __device__ constexpr int tiled_ring_bytes() {
  return NS * KD * (BM + BN) / 16 * 1024;
}
template <int EPI, int BM, int BN, int KD, int NS>
__host__ __device__ constexpr int tiled_lds_bytes() {
  return tiled_ring_bytes<BM, BN, KD, NS>() + (ln_on_load<EPI>() ? BM * 8 : 0);
}

// One kilobyte from a buffer straight into LDS: lane offset voff, wave-uniform
// offset soff + pos, LDS byte address slot + dst.  Inline asm, so that the
// compiler does not see an LDS write: it would wait for every outstanding one
// before any LDS read (it cannot tell the ring's slots apart) and empty the
// ring.  No vector register is written; the kernel counts these loads itself.
// Nor does the compiler see a memory instruction that reads scalar registers,
// so the wait states that it would put before one are here: five after a vector
// instruction that wrote one of them (v_readlane of a spilled register,
// v_readfirstlane), which covers the one after the write of M0.  The two
// additions are two of them and s_nop 2 is three; the sum that the load reads is
// written by the scalar unit, which needs none.
__device__ __forceinline__ void stage_kb(const u32x4_t& rsrc, uint32_t voff, uint32_t soff, uint32_t pos, uint32_t slot,
                                         uint32_t dst) {
  uint32_t off;
  asm volatile(
      "s_add_u32 m0, %1, %2\n\ts_add_u32 %0, %3, %4\n\ts_nop 2\n\tbuffer_load_dwordx4 %5, %6, %0 offen lds"
      : "=&s"(off)
      : "s"(slot), "s"(dst), "s"(soff), "s"(pos), "v"(voff), "s"(rsrc)
      : "m0", "scc");
}
__device__ __forceinline__ void compiler_fence() { asm volatile("" ::: "memory"); }

// Slots that the staging runs ahead of the products.  One barrier per slot, in
// its last step: behind the barrier of slot q every wave has multiplied, and so
// read, slot q - 1 to the end, and may still be reading slot q.  The staging of
// a slot's first step refills the slot that is free then: q - 1 when that step
// is behind the barrier (a slot of one step), else q - 2.
template <int BM, int WR, int KD, int NS>
__host__ __device__ constexpr int tiled_ahead() {
  static_assert(NS >= 3, "a slot being read, one landing and one being refilled");
  return KD == 1 && BM / 16 / WR <= 4 ? NS - 1 : NS - 2;
}

// workgroups that a CU holds (its LDS is 160 KB; with two, 128 registers a lane)
template <int EPI, int BM, int BN, int KD, int NS>
__host__ __device__ constexpr int tiled_per_cu() {
  return tiled_lds_bytes<EPI, BM, BN, KD, NS>() <= 81920 ? 2 : 1;
}

template <int EPI, int BM, int BN, int WR, int KD, int NS>
__global__ __launch_bounds__(512, (2 * tiled_per_cu<EPI, BM, BN, KD, NS>())) void gemm_tiled_kernel(GemmArgs a) {
  using T = uint16_t;
  constexpr int WC = kTiledWaves / WR;
  constexpr int TRB = BM / 16, CBB = BN / 16;          // row tiles, column blocks per workgroup
  constexpr int FPC = TRB + CBB, FPS = FPC * KD;       // fragments per chunk, per slot
  constexpr int LA = TRB * KD / kTiledWaves, LW = CBB * KD / kTiledWaves;  // fragment loads per wave and slot
  static_assert(LA * kTiledWaves == TRB * KD && LW * kTiledWaves == CBB * KD, "every wave stages as many fragments");
  constexpr int LPW = LA + LW;
  constexpr int TR = TRB / WR, TC = CBB / WC;          // per wave
  constexpr bool LNA = ln_on_load<EPI>();
  // A slot is multiplied in S steps of H row tiles x TC column blocks of one
  // chunk.  The fragments of a step are read while the step before it is
  // multiplied, into the other of two register sets (W: per chunk).
  constexpr int H = TR > 4 ? TR / 2 : TR, HS = TR / H, S = HS * KD;
  constexpr int AHEAD = tiled_ahead<BM, WR, KD, NS>();
  static_assert(AHEAD == (S == 1 ? NS - 1 : NS - 2), "see tiled_ahead");
  extern __shared__ __align__(16) char smem[];
  float2* s_ps = reinterpret_cast<float2*>(smem + tiled_ring_bytes<BM, BN, KD, NS>());  // [BM] (sum, sum of squares)

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int wr = w / WC, wc = w % WC;
  const int D = a.sh.D;
  const int M = a.meta->m;
  const int nblocks = a.Nout / 16, kchunks = a.kchunks, akc = a.lda / 32;
  const int mt = (M + BM - 1) / BM, nt = (nblocks + CBB - 1) / CBB;  // tiles that have rows
  const int per_split = mt * nt, total = per_split * a.ksplit;
  const int kper = (kchunks + a.ksplit - 1) / a.ksplit;
  // groups of GM row tiles, column-major inside a group: an XCD's contiguous
  // range of positions is a compact block of tiles
  const int GM = max(1, min(a.rgroups, mt));

  struct Tile {
    int m0, cb0, ks, kbeg, nk;  // nk: chunks
  };
  // the i-th tile of this workgroup, i < its count of tiles.  The hardware
  // deals workgroups to the 8 XCDs round robin (the grid is a multiple of 8 or
  // one workgroup per tile), so index % 8 is the XCD; each XCD is given a
  // contiguous range of positions.
  auto tile_of = [&](int idx) {
    const int xcd = idx % 8, per = total / 8, rem = total % 8;
    int pos = xcd * per + min(xcd, rem) + idx / 8;
    Tile t;
    t.ks = pos / per_split;
    pos -= t.ks * per_split;
    const int grp = pos / (GM * nt), inside = pos - grp * GM * nt;
    const int gm = min(GM, mt - grp * GM);
    t.m0 = (grp * GM + inside % gm) * BM;
    t.cb0 = (inside / gm) * CBB;
    t.kbeg = t.ks * kper;
    t.nk = min(kchunks - t.kbeg, kper);
    return t;
  };
  const int stride = gridDim.x;
  if ((int)blockIdx.x >= total) return;  // uniform

  // Staging.  A row tile t, chunk kc is kilobyte t * akc + kc of the compact
  // rows; W column block b, chunk kc kilobyte b * kchunks + kc of the packed
  // weights; fragment (sub-chunk s, r) of a slot sits at (s * FPC + r) KB, A
  // first.  A row tile, column block or chunk past its operand's end stages the
  // last one instead, whose products are skipped or never stored.  The stream
  // of slots runs AHEAD ahead of the products and on into the workgroup's next
  // tile (the launch gives a workgroup several tiles only if each has more than
  // AHEAD slots, so that the tile after the staged one is known when it ends);
  // past the last tile the resources' sizes are zero, so the loads move nothing
  // and every slot still counts LPW loads: the K loop has neither branches nor
  // wait counts that depend on the position.
  auto rsrc_of = [](const void* p, uint32_t bytes) {
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    return u32x4_t{(uint32_t)b, (uint32_t)(b >> 32) & 0xffffu, bytes, 0x00020000u};
  };
  const uint32_t sizeA = (uint32_t)a.mpad * a.lda * 2, sizeW = (uint32_t)nblocks * kchunks * 1024;
  u32x4_t rA = rsrc_of(a.A, sizeA), rW = rsrc_of(a.W, sizeW);
  const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
  const int atiles = a.mpad / 16;
  constexpr uint32_t SLOT = FPS * 1024, RING = NS * SLOT, STEP = KD * 1024;
  struct Src {  // byte offsets of this wave's fragments of a tile's first slot; the tile's chunks in bytes
    uint32_t a[LA], w[LW], end;
  };
  auto src_of = [&](int idx) {
    const Tile t = tile_of(idx);
    Src r;
#pragma unroll
    for (int j = 0; j < LA; ++j)
      r.a[j] = (uint32_t)(min(t.m0 / 16 + (w + kTiledWaves * j) % TRB, atiles - 1) * akc + t.kbeg) * 1024;
#pragma unroll
    for (int j = 0; j < LW; ++j)
      r.w[j] = (uint32_t)(min(t.cb0 + (w + kTiledWaves * j) % CBB, nblocks - 1) * kchunks + t.kbeg) * 1024;
    r.end = (uint32_t)t.nk * 1024;
    return r;
  };
  auto dst_of = [&](int f, int per, int first) {  // LDS offset of fragment f within a slot
    return (uint32_t)((f / per) * FPC + first + f % per) * 1024;
  };
  const uint32_t voff = lane * 16;
  Src cur = src_of(blockIdx.x), nxt;
  uint32_t nsizeA, nsizeW;
  auto set_next = [&](int idx) {  // uniform: the tile after idx
    const bool any = idx + stride < total;
    nxt = any ? src_of(idx + stride) : cur;
    nsizeA = any ? sizeA : 0;
    nsizeW = any ? sizeW : 0;
  };
  set_next(blockIdx.x);
  uint32_t ipos = 0, islot = ring_lds;
  auto stage_one = [&](int j) {  // load j (compile time) of this wave's LPW for the next slot of the stream
    const bool isA = j < LA;
    const int f = w + kTiledWaves * (isA ? j : j - LA), per = isA ? TRB : CBB;
    const uint32_t pos = KD == 1 ? ipos : min(ipos + (uint32_t)(f / per) * 1024, cur.end - 1024);
    if (isA) stage_kb(rA, voff, cur.a[isA ? j : 0], pos, islot, dst_of(f, TRB, 0));
    else stage_kb(rW, voff, cur.w[isA ? 0 : j - LA], pos, islot, dst_of(f, CBB, TRB));
  };
  auto staged = [&]() {  // all of them are issued
    ipos += STEP;
    islot += SLOT;
    islot = islot == ring_lds + RING ? ring_lds : islot;
    const bool wrap = ipos >= cur.end;  // uniform: selects, no branch
#pragma unroll
    for (int j = 0; j < LA; ++j) cur.a[j] = wrap ? nxt.a[j] : cur.a[j];
#pragma unroll
    for (int j = 0; j < LW; ++j) cur.w[j] = wrap ? nxt.w[j] : cur.w[j];
    rA.z = wrap ? nsizeA : rA.z;
    rW.z = wrap ? nsizeW : rW.z;
    cur.end = wrap ? nxt.end : cur.end;
    ipos = wrap ? 0 : ipos;
  };
#pragma unroll
  for (int c = 0; c < AHEAD; ++c) {
#pragma unroll
    for (int j = 0; j < LPW; ++j) stage_one(j);
    staged();
  }
  const uint32_t offA = (uint32_t)(wr * TR) * 1024 + lane * 16;
  const uint32_t offW = (uint32_t)(TRB + wc * TC) * 1024 + lane * 16;
  uint32_t rslot = 0;  // byte offset of the slot being multiplied
  // LayerNorm statistics: of a step's H row tiles each wave sums SH (wave
  // columns beyond H repeat another's)
  constexpr int SH = LNA ? (H > WC ? H / WC : 1) : 0, SHA = SH > 0 ? SH : 1;
  static_assert(!LNA || H % WC == 0 || WC % H == 0, "a step's row tiles split evenly over the wave columns");
  const uint32_t offS = (uint32_t)(wr * TR + wc % H) * 1024 + lane * 16;
  u32x4_t af[2][H], wf[2][TC], sf[2][SHA];
  // read k of the TC + H + SH (without the W fragments H + SH) fragments of step (slot, sub, half)
  auto read_one = [&](int k, bool neww, u32x4_t (&fa)[H], u32x4_t (&fw)[TC], u32x4_t (&fs)[SHA], uint32_t slot, int sub,
                      int half) {
    const int kw = neww ? TC : 0;
    auto at = [&](uint32_t off, int frag) { return *reinterpret_cast<const u32x4_t*>(smem + (slot + off) + frag * 1024); };
    if (k < kw) fw[k < TC ? k : 0] = at(offW, sub * FPC + k);
    else if (k < kw + H) fa[(k - kw) % H] = at(offA, sub * FPC + half * H + k - kw);
    else fs[(k - kw - H) % SHA] = at(offS, sub * FPC + half * H + (k - kw - H) * WC);
  };
  // The slot after `rslot` may be read once every wave's share of it has
  // landed: each wave waits until at most the loads of the slots issued after
  // it are outstanding (they complete in order), then the barrier.
  auto advance = [&]() {
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(LPW * (NS - 3)));
    compiler_fence();
    __builtin_amdgcn_s_barrier();
    compiler_fence();
    rslot += SLOT;
    rslot = rslot == RING ? 0 : rslot;
  };

  // the first slot, and its first step's fragments
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(LPW * (AHEAD - 1)));
  __builtin_amdgcn_s_barrier();
  compiler_fence();
#pragma unroll
  for (int k = 0; k < TC + H + SH; ++k) read_one(k, true, af[0], wf[0], sf[0], 0, 0, 0);

  for (int idx = blockIdx.x; idx < total; idx += stride) {
    const Tile t = tile_of(idx);
    if (idx != (int)blockIdx.x) set_next(idx);
    f32x4_t acc[TR][TC];
#pragma unroll
    for (int r = 0; r < TR; ++r)
#pragma unroll
      for (int b = 0; b < TC; ++b) acc[r][b] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4_t accs[HS * SHA], accq[HS * SHA];  // row sums and sums of squares (LNA)
#pragma unroll
    for (int i = 0; i < HS * SHA; ++i) accs[i] = accq[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    V8<T> one;
    ones(one);

    // no scalar load is left in flight: with one the compiler could not count
    // LDS reads in the loop and would wait for all of them
    __builtin_amdgcn_s_waitcnt(lgkmcnt0_imm());
    // one slot; PA, PW: the register sets that hold its first step
    auto slot_steps = [&](int kc, auto pa_, auto pw_) {
      constexpr int PA = decltype(pa_)::value, PW = decltype(pw_)::value;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int sub = s / HS, half = s % HS, ca = (PA + s) & 1, cw = (PW + sub) & 1;
        const bool last = s + 1 == S, neww = last || (s + 1) % HS == 0;
        const int nsub = last ? 0 : (s + 1) / HS, nhalf = last ? 0 : (s + 1) % HS;
        if (last) advance();
        // The next step's reads and (in the slot's first step) the staging are
        // spread over the row tiles' products, which they run beside: issued
        // together they would hold up the products behind them.
        const int reads = (neww ? TC : 0) + H + SH;
        const bool run = sub == 0 || kc + sub < t.nk;  // uniform
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < H; ++i) {
          if (run) {
            V8<T> x;
            x.v = __builtin_bit_cast(uint4, af[ca][i]);
#pragma unroll
            for (int b = 0; b < TC; ++b) {
              V8<T> y;
              y.v = __builtin_bit_cast(uint4, wf[cw][b]);
              mma(acc[half * H + i][b], y, x);
            }
          }
#pragma unroll
          for (int k = 0; k < TC + H + SH; ++k)
            if (k >= reads * i / H && k < reads * (i + 1) / H)
              read_one(k, neww, af[ca ^ 1], wf[cw ^ 1], sf[ca ^ 1], rslot, nsub, nhalf);
          if (s == 0) {
#pragma unroll
            for (int j = 0; j < LPW; ++j)
              if (j >= LPW * i / H && j < LPW * (i + 1) / H) stage_one(j);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (s == 0) staged();
        if (run) {
#pragma unroll
          for (int i = 0; i < SH; ++i) {
            V8<T> x;
            x.v = __builtin_bit_cast(uint4, sf[ca][i]);
            mma(accs[half * SHA + i], x, one);
            mma(accq[half * SHA + i], x, x);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, S & 1>;
    using C2 = std::integral_constant<int, KD & 1>;
    if constexpr (S % 2 == 0 && KD % 2 == 0) {
      for (int kc = 0; kc < t.nk; kc += KD) slot_steps(kc, C0{}, C0{});
    } else {
      // pairs of slots, so that every register set is known at compile time;
      // an odd one first, its sets moved back
      int kc = 0;
      if ((t.nk + KD - 1) / KD % 2) {
        slot_steps(0, C0{}, C0{});
        if constexpr (S % 2 == 1) {
#pragma unroll
          for (int i = 0; i < H; ++i) af[0][i] = af[1][i];
#pragma unroll
          for (int i = 0; i < SH; ++i) sf[0][i] = sf[1][i];
        }
#pragma unroll
        for (int b = 0; b < TC; ++b) wf[0][b] = wf[1][b];
        kc = KD;
      }
      for (; kc < t.nk; kc += 2 * KD) {
        slot_steps(kc, C0{}, C0{});
        slot_steps(kc + KD, C1{}, C2{});
      }
    }

    // ---- LayerNorm statistics: lane (g, n) holds rows 4g..4g+3 of column n, so
    // row n's sum (any column) and sum of squares (the diagonal) are element
    // n - 4g
    float rstd[TR], nmr[TR];
    if constexpr (LNA) {
#pragma unroll
      for (int i = 0; i < HS * SHA; ++i) {
        const int r = (i / SHA) * H + wc % H + (i % SHA) * WC, e = n - 4 * g;
        if (e >= 0 && e < 4) s_ps[(wr * TR + r) * 16 + n] = make_float2(elem4(accs[i], e), elem4(accq[i], e));
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      compiler_fence();
#pragma unroll
      for (int r = 0; r < TR; ++r) {
        const float2 p = s_ps[(wr * TR + r) * 16 + n];
        const float mean = p.x / (float)D;
        const float var = fmaxf(p.y / (float)D - mean * mean, 0.0f);
        rstd[r] = 1.0f / sqrtf(var + a.sh.eps);
        nmr[r] = -mean * rstd[r];
      }
    }

    // ---- epilogue: lane (g, n) holds columns 4g..4g+3 of row n of each 16x16
    // tile.  Operations and rounding points are the small-M kernel's
    // (epilogue_store).  The rows' map entries are loaded once, and a column
    // block's operands while the block before it is finished: loaded where
    // they are used, behind the masked stores, every one of them would wait
    // out its latency.  Loads and arithmetic run for every lane (rows past M
    // take the last row's operands) and only the stores are masked, so no load
    // is left unwaited on any path and the compiler puts no wait for one into
    // the K loop.
    const int ldk = a.ldo / 32;
    RowInfo rinfo[TR];
#pragma unroll
    for (int r = 0; r < TR; ++r) {
      rinfo[r] = RowInfo{nullptr, 0, 0};
      if constexpr (has_rows<EPI>()) rinfo[r] = a.rows[min(t.m0 + (wr * TR + r) * 16 + n, M - 1)];
    }
    struct ColOps {
      float4 bias, c1;
      uint2 res[TR];
    } ops[2];
    auto load_ops = [&](ColOps& q, int b) {
      const int col = min(t.cb0 + wc * TC + b, nblocks - 1) * 16 + 4 * g;
      if constexpr (EPI != EPI_PART) q.bias = *reinterpret_cast<const float4*>(a.bias + col);
      if constexpr (LNA) q.c1 = *reinterpret_cast<const float4*>(a.c1 + col);
      if constexpr (has_resid<EPI>()) {
#pragma unroll
        for (int r = 0; r < TR; ++r)
          q.res[r] = *reinterpret_cast<const uint2*>(static_cast<const T*>(a.resid) +
                                                     frag_row(min(t.m0 + (wr * TR + r) * 16 + n, M - 1), ldk) + frag_col(col));
      }
    };
    load_ops(ops[0], 0);
    if constexpr (has_rows<EPI>()) {
#pragma unroll
      for (int r = 0; r < TR; ++r) asm volatile("" : "+v"(rinfo[r].cache), "+v"(rinfo[r].tok));
    }
#pragma unroll
    for (int b = 0; b < TC; ++b) {
      if (b + 1 < TC) load_ops(ops[(b + 1) & 1], b + 1);
      const ColOps& q = ops[b & 1];
      const int cb = t.cb0 + wc * TC + b;
      const int col = min(cb, nblocks - 1) * 16 + 4 * g;
      const float bv[4] = {q.bias.x, q.bias.y, q.bias.z, q.bias.w}, cv[4] = {q.c1.x, q.c1.y, q.c1.z, q.c1.w};
      size_t cpart = 0;
      int which = 0;  // uniform: a block never straddles Q, K, V (D % 16 == 0)
      if constexpr (EPI == EPI_QKV) {
        which = min(cb, nblocks - 1) * 16 / D;
        const int c = col - which * D, hh = c / a.sh.dh, d = c - hh * a.sh.dh;  // dh % 8 == 0: one head
        cpart = which == 0 ? (size_t)c : which == 1 ? k_col(a.sh, hh, d) : v_col(a.sh, hh, d);
      } else if constexpr (EPI == EPI_RES || EPI == EPI_DOWN || EPI == EPI_FC1) {
        cpart = frag_col(col);
      } else {
        cpart = (size_t)col;
      }
#pragma unroll
      for (int r = 0; r < TR; ++r) {
        const int row = t.m0 + (wr * TR + r) * 16 + n;
        const bool ok = row < M && cb < nblocks;
        const f32x4_t x = acc[r][b];
        const size_t rpart = frag_row(row, ldk);
        float o[4];
        if constexpr (EPI == EPI_PART) {
          if (ok)
            *reinterpret_cast<float4*>(static_cast<float*>(a.out) + ((size_t)t.ks * a.mpad + row) * a.ldo + cpart) =
                make_float4(x[0], x[1], x[2], x[3]);
          continue;
        } else if constexpr (EPI == EPI_RES || EPI == EPI_DOWN) {  // S(resid + S(x + b))
          const uint2 rv = q.res[r];
          const float res[4] = {__uint_as_float(rv.x << 16), __uint_as_float(rv.x & 0xffff0000u),
                                __uint_as_float(rv.y << 16), __uint_as_float(rv.y & 0xffff0000u)};
#pragma unroll
          for (int j = 0; j < 4; ++j) o[j] = res[j] + Elem<T>::rnd(x[j] + bv[j]);
        } else if constexpr (EPI == EPI_ATT) {
#pragma unroll
          for (int j = 0; j < 4; ++j) o[j] = x[j] + bv[j];
        } else if constexpr (EPI == EPI_QKV) {
#pragma unroll
          for (int j = 0; j < 4; ++j) o[j] = fmaf(rstd[r], x[j], fmaf(nmr[r], cv[j], bv[j]));
        } else {  // EPI_FC1
#pragma unroll
          for (int j = 0; j < 4; ++j) o[j] = gelu_tanh(Elem<T>::rnd(fmaf(rstd[r], x[j], fmaf(nmr[r], cv[j], bv[j]))));
        }
        u32x2_t ov = {f2bf2(o[0], o[1]), f2bf2(o[2], o[3])};
        asm volatile("" : "+v"(ov));
        if (!ok) continue;
        auto put = [&](T* p) { *gbl(reinterpret_cast<u32x2_t*>(p)) = ov; };
        if constexpr (EPI == EPI_RES || EPI == EPI_DOWN || EPI == EPI_FC1) {
          put(static_cast<T*>(a.out) + rpart + cpart);
          if constexpr (EPI == EPI_DOWN) put(x_row<T>(rinfo[r].cache, a.cl, a.sh, a.layer + 1, rinfo[r].tok) + col);
        } else if constexpr (EPI == EPI_ATT) {
          put(reinterpret_cast<T*>(rinfo[r].cache + a.cl.a + (size_t)a.layer * a.cl.x_layer) + (size_t)rinfo[r].tok * D + cpart);
        } else if constexpr (EPI == EPI_QKV) {
          if (which == 0) {
            put(static_cast<T*>(a.out) + (size_t)row * a.ldo + cpart);
          } else if (which == 1) {  // K: consecutive dims are contiguous
            put(reinterpret_cast<T*>(rinfo[r].cache + a.cl.k + (size_t)a.layer * a.cl.kv_layer) + k_tok(a.sh, rinfo[r].tok) + cpart);
          } else {  // V (transposed): consecutive dims are 8 elements apart
            T* vb = reinterpret_cast<T*>(rinfo[r].cache + a.cl.v + (size_t)a.layer * a.cl.kv_layer) + v_tok(a.sh, rinfo[r].tok) + cpart;
#pragma unroll
            for (int j = 0; j < 4; ++j) gbl(vb)[8 * j] = f2bf(o[j]);
          }
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // no load into this workgroup's LDS outlives it
}

template <int EPI, int BM, int BN, int WR, int KD, int NS>
hipError_t launch_tiled_cfg(const GemmArgs& a, int rows, hipStream_t s) {
  constexpr int lds = tiled_lds_bytes<EPI, BM, BN, KD, NS>();
  if constexpr (lds > 65536) {
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tiled_kernel<EPI, BM, BN, WR, KD, NS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (attr != hipSuccess) return attr;
  }
  constexpr int slots = 256 * tiled_per_cu<EPI, BM, BN, KD, NS>();  // workgroups the chip holds
  const int mt = (rows + BM - 1) / BM, nt = (a.Nout + BN - 1) / BN;
  const int total = mt * nt * a.ksplit;
  // row tiles per group: about the square root of one XCD's share of the tiles
  // at work together, at most mt
  GemmArgs b = a;
  const int per_xcd = (std::min(total, slots) + 7) / 8;
  int gm = 1;
  while ((gm + 1) * (gm + 1) * BM <= per_xcd * BN) ++gm;
  b.rgroups = std::max(1, std::min(gm, mt));
  // several tiles to a workgroup only if each has more slots than the staging
  // runs ahead
  const int kper = (a.kchunks + a.ksplit - 1) / a.ksplit, klast = a.kchunks - kper * (a.ksplit - 1);
  const bool shared = (std::min(kper, klast) + KD - 1) / KD > tiled_ahead<BM, WR, KD, NS>();
  return launch_k(gemm_tiled_kernel<EPI, BM, BN, WR, KD, NS>, dim3(shared ? std::min(total, slots) : total), dim3(512),
                  (size_t)lds, s, b);
}

// The tile by the number of tiles that it gives, on 256 CUs.  `expected` is the
// row count to tune for, `rows` the most that the call can have (they differ
// when M is only known on the device; the kernel reads it).  us per launch on
// weights from HBM, So400m (D 1152, F 4304) or ViT-L (D 1024, F 4096) widths:
//   64 x 64 (one per CU, 128 KB ring) while it gives at most one tile per CU,
//     then 64 x 128 while that does: what a CU can stage bounds them, so the
//     smaller of the two that fits one round is the faster: QKV of 256 rows 9.9
//     (64 x 128: 11.7), MLP up of 256 rows 11.9 (64 x 64: 14.0), output
//     projection of 1024 rows 9.0 (64 x 64: 10.5, 128 x 128: 12.3), MLP down of
//     2048 rows 23.7 (128 x 128: 32);
//   256 x 256 for the widest products (QKV, MLP up) where its tiles are a
//     multiple of the CUs: MLP up of 8192 rows, 512 tiles, 77 (256 x 128: 95,
//     128 x 128: 93), QKV of 16384 rows, 768 tiles, 110 (256 x 128: 129); QKV of
//     8192 rows, 384 tiles in two rounds, 73 (256 x 128: 71); the numbers in
//     between are not measured;
//   256 x 128 where it gives more than half a tile per CU and one round, or
//     rounds that are full to three quarters on the whole: MLP down of 8192 rows
//     63 (128 x 128: 75), QKV of 8192 rows, 384 tiles in two rounds of 256, 71
//     (74), MLP up of 1024 rows 22.4 (24.4);
//   128 x 128 for the rest: QKV of 1024 rows 15.8 (64 x 128: 20), MLP up of
//     512 rows 14.9 (64 x 128: 19.3); with at most one per CU its ring takes
//     the whole LDS, more ahead of weights that come from HBM: QKV of 1024
//     rows within the 448x448 encode 20.1 -> 17.6; else two per CU.
template <int EPI>
hipError_t launch_tiled_epi(const GemmArgs& a, int expected, int rows, hipStream_t s) {
  if (!a.sh.dtype || a.ksplit < 1 || a.sh.dh % 8) return hipErrorInvalidValue;
  if (a.ksplit > 1) {
    const int kper = (a.kchunks + a.ksplit - 1) / a.ksplit;
    if (EPI != EPI_PART || kper * (a.ksplit - 1) >= a.kchunks) return hipErrorInvalidValue;
  }
  auto tiles = [&](int bm, int bn) { return (expected + bm - 1) / bm * ((a.Nout + bn - 1) / bn) * a.ksplit; };
  if (tiles(64, 64) <= 256) return launch_tiled_cfg<EPI, 64, 64, 2, 2, 8>(a, rows, s);
  if (tiles(64, 128) <= 256) return launch_tiled_cfg<EPI, 64, 128, 2, 2, 6>(a, rows, s);
  // at least `quarters` quarters of the places in all rounds of t tiles
  auto full = [](int t, int quarters) { return 4 * t >= quarters * 256 * ((t + 255) / 256); };
  if constexpr (EPI == EPI_QKV || EPI == EPI_FC1) {
    const int x = tiles(256, 256);
    if (x >= 256 && full(x, 4)) return launch_tiled_cfg<EPI, 256, 256, 2, 1, 4>(a, rows, s);
  }
  const int l = tiles(256, 128);
  if (l > 128 && (l <= 256 || full(l, 3))) return launch_tiled_cfg<EPI, 256, 128, 4, 1, 6>(a, rows, s);
  if (tiles(128, 128) <= 256) return launch_tiled_cfg<EPI, 128, 128, 2, 1, 8>(a, rows, s);
  return launch_tiled_cfg<EPI, 128, 128, 2, 1, 4>(a, rows, s);
}

}  // namespace incvit
