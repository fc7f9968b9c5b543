// Attention forward O = softmax(scale * Q K^T [+ causal mask]) V for gfx950 when the query rows alone
// do not fill the chip: the keys are split over groups of wavefronts inside the workgroup.
//
// The same FlashAttention-2 recurrence and transposed products as mha_pp.hip (arXiv 2503.14985,
// Section 2.5, Algorithm 1), with the warp distribution the paper gives its paged kernel (Section 3.2,
// Listing 6): a workgroup of 8 wavefronts owns 32 * QW query rows (QW = 2 or 4 wavefronts side by side)
// and KW = 8 / QW groups of them take every KW-th key tile, each group with its own running maximum,
// sum and output; the groups' results meet once, in LDS, at the end. The 256-row workgroups of
// mha_pp.hip leave most of the chip idle when batch * heads * ceil(Sq / 256) is small and walk all keys
// one tile after the other; here there are 2 to 4 times as many workgroups for the same problem, or (few
// query rows) as many that each take a quarter of the time.
//
// Schedule. Per key tile (32 keys) a wavefront does X_t, the softmax of S_t on the vector ALU, and C_t,
// the MFMAs O^T += V_t^T P_t^T and S_{t+1}^T = K_{t+1} Q^T. Between two workgroup barriers (interval t)
// wavefronts 0-3 run C_t, X_{t+1} and wavefronts 4-7, the other half of every SIMD, X_t, C_t: one does
// matrix work while the other one does exponentials.
//
// A group's tiles go straight into LDS, in the order in which they are read, s_0 = K_0, s_1 = K_1, s_2 = V_0,
// s_3 = K_2, s_4 = V_1, ...: interval t reads s_{2t+1} and s_{2t+2}. They sit in a ring of R slots (s_i in slot
// i % R), so interval t can fetch s_{2t+R-1} and s_{2t+R} into the slots it finds free.
//
// What bounds it: one interval, 0.7 to 0.8 us, is the serial path of a wavefront through a 32-key tile (512
// clocks of MFMA for D = 128, about as much of vector ALU work, the latency of the first V fragments behind
// the barrier); the LDS has no room for tiles of 64 keys for four groups. 2 x 16 heads, 333 x 1501, D = 128:
// 36.3 us on the 256-row kernel, 20.3 here; 1 x 8 heads, 200 x 1000, D = 64: 20.4 -> 11.2. With checks of
// what is left to do in every interval instead of a loop of its own for the full ones 22.5, with one
// fragment read, awaited and multiplied at a time 24.
#include <type_traits>

#include "mha_tile.h"
#include "mlt_internal.h"

namespace mlt {

namespace {

template <int D, int QW> struct KsCfg {
  static constexpr int KW = 8 / QW;                // key groups
  static constexpr int KEYS = 32;                  // keys per tile
  static constexpr int BM = 32 * QW;               // query rows per workgroup
  static constexpr int ROWB = D * 2;
  static constexpr int TILE_B = KEYS * ROWB;       // one K or V tile = one slot
  static constexpr int R = QW == 2 ? 5 : 10;       // slots per group: 160 KB in all, 80 KB for D = 64 (two workgroups per CU)
  static constexpr int SMEM = KW * R * TILE_B;
  static constexpr int PSTR = D + 4;               // floats per parked output row (16-byte aligned, rows in different banks)
  static constexpr int STAT_OFF = 8 * 32 * PSTR * 4;   // parked outputs, then maxima and sums, over the ring once that is done with
  static_assert(STAT_OFF + 8 * 32 * 2 * 4 <= SMEM, "the parking area");
  static constexpr int CPR = D / 8, RPB = 64 / CPR;        // 16-byte chunks per row, rows per 1 KB load
  static constexpr int LPW = KEYS / RPB / QW;              // loads per wavefront and tile
  static constexpr int NKK = D / 16, NDT = D / 32;
};

// O (SPLIT = false), or, when blockIdx.y selects one of gridDim.y ranges of the key tiles, that range's
// fp32 partial result: outputs not yet divided by the sum, po[range][row][D], and maximum (log2
// domain) and sum, ps[range][row][2], with `row` counting all batch * heads * Sq rows.
template <typename Tag, int D, int QW, bool SPLIT, bool CAUSAL>
__global__ __launch_bounds__(512, D == 64 ? 4 : 2) void mha_ks_kernel(
    const uint16_t* __restrict__ Q, const uint16_t* __restrict__ K, const uint16_t* __restrict__ V,
    uint16_t* __restrict__ O, float* __restrict__ po, float* __restrict__ ps, int Sq, int Sk, int nq,
    int total, int nxcd, float c, int negate, MaskedMap map) {
  typedef KsCfg<D, QW> L;
  typedef PaCfg<D> P;                              // swizzles
  typedef typename Elem<Tag>::vec8 V8;
  constexpr int KW = L::KW, R = L::R, ROWB = L::ROWB, NKK = L::NKK, NDT = L::NDT;
  extern __shared__ __align__(16) char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave % QW, kg = wave / QW;
  const bool late = wave >= 4;                     // the half of a SIMD's wavefronts that runs X before C
  const int lq = lane & 31, h = lane >> 5;
  int bh, qt;
  if (CAUSAL && map.chunk > 0) block_map_masked(blockIdx.x, nq, nxcd, map, bh, qt);
  else block_map(blockIdx.x, total, nq, CAUSAL ? nxcd & 255 : nxcd, bh, qt);
  const int q0 = qt * L::BM + qw * 32;             // first query row of this wavefront
  const int my_q = q0 + lq;

  const uint16_t* Qh = Q + (int64_t)bh * Sq * D;
  const char* Kh = reinterpret_cast<const char*>(K + (int64_t)bh * Sk * D);
  const char* Vh = reinterpret_cast<const char*>(V + (int64_t)bh * Sk * D);

  // key tiles of this workgroup: those its last query row sees (all without the mask), or a range of them
  int kv_len = Sk;
  if (CAUSAL) {
    const int last_q = (qt + 1) * L::BM < Sq ? (qt + 1) * L::BM : Sq;     // exclusive
    kv_len = last_q < Sk ? last_q : Sk;
  }
  int tb = 0, te = (kv_len + L::KEYS - 1) / L::KEYS;
  if (SPLIT) {
    const int all = (Sk + L::KEYS - 1) / L::KEYS, per = (all + (int)gridDim.y - 1) / (int)gridDim.y;
    tb = (int)blockIdx.y * per;
    te = tb + per < te ? tb + per : te;
  }
  const int T = te > tb ? (te - tb + KW - 1) / KW : 0;             // steps of the workgroup
  const int Tg = te - tb > kg ? (te - tb - kg + KW - 1) / KW : 0;   // tiles of this key group: tb + kg + t * KW
  // steps in which this wavefront has visible keys, and from which one of them on a score has to be
  // masked (causal, or the last tile reaches past Sk)
  int Tw = q0 < Sq ? Tg : 0;
  int t_mask = Tg - 1 >= 0 && (tb + kg + (Tg - 1) * KW + 1) * L::KEYS > Sk ? Tg - 1 : Tg;
  if (CAUSAL) {
    const int last = (q0 + 31) / L::KEYS - tb - kg;                // tiles up to the one of this wavefront's last row
    const int vis = last >= 0 ? last / KW + 1 : 0;
    Tw = Tw < vis ? Tw : vis;
    const int first = (q0 + 1) / L::KEYS - tb - kg;                // tiles from here on reach past its first row
    const int tm = first > 0 ? (first + KW - 1) / KW : 0;
    t_mask = t_mask < tm ? t_mask : tm;
  }
  const int t_ragged = Tg - 1 >= 0 && (tb + kg + (Tg - 1) * KW + 1) * L::KEYS > Sk ? Tg - 1 : -1;

  V8 qf[NKK];                                      // as in mha_pp_kernel
  {
    const int row = my_q < Sq ? my_q : Sq - 1;
    const uint16_t* qp = Qh + (int64_t)row * D + 8 * h;
    const uint32_t flip = negate ? 0x80008000u : 0u;
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) {
      u32x4 raw = *reinterpret_cast<const u32x4_mem*>(qp + kk * 16);
      raw[0] ^= flip; raw[1] ^= flip; raw[2] ^= flip; raw[3] ^= flip;
      qf[kk] = __builtin_bit_cast(V8, raw);
    }
  }

  // ---- global -> LDS: wavefront qw of a key group fills blocks qw*LPW .. of the group's tiles
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
  const uint32_t grp0 = lds0 + kg * (R * L::TILE_B);
  uint32_t voff_k[L::LPW], voff_v[L::LPW];
#pragma unroll
  for (int i = 0; i < L::LPW; ++i) {
    const int row = (qw * L::LPW + i) * L::RPB + lane / L::CPR;
    voff_k[i] = (uint32_t)row * ROWB + (uint32_t)((lane % L::CPR) ^ P::fk(row)) * 16u;
    voff_v[i] = (uint32_t)row * ROWB + (uint32_t)((lane % L::CPR) ^ P::fv(row)) * 16u;
  }
  // K or V tile of this group's t-th step into ring slot `slot`
  auto issue = [&](int t, const char* base, const uint32_t (&voff)[L::LPW], int slot) __attribute__((always_inline)) {
    if (t >= Tg) return;
    const int n = tb + kg + t * KW;
    const char* gp = base + (int64_t)n * L::TILE_B;
    const uint32_t dst = grp0 + slot * L::TILE_B + qw * (L::LPW * 1024);
    if (t != t_ragged) {
#pragma unroll
      for (int i = 0; i < L::LPW; ++i) load_lds16(gp, voff[i], dst + i * 1024);
    } else {
      // rows past Sk re-read row Sk-1 (their weights are forced to 0)
      const int last = Sk - 1 - n * L::KEYS;
#pragma unroll
      for (int i = 0; i < L::LPW; ++i) {
        const int row = (qw * L::LPW + i) * L::RPB + lane / L::CPR;
        load_lds16(gp, voff[i] - (row > last ? (uint32_t)(row - last) * ROWB : 0u), dst + i * 1024);
      }
    }
  };

  // ---- fragment addresses inside a slot: as in mha_pp_kernel
  const int k_frag = lq * ROWB + ((h ^ P::fk(lq)) << 4);
  const int vg = lane >> 4, vs = lane & 15;
  const int v_row = 4 * (vg >> 1) + (vs >> 2);
  const int v_frag = v_row * ROWB + (((2 * (vg & 1) + ((vs & 3) >> 1)) ^ P::fv(v_row)) << 4) + 8 * (vs & 1);

  f32x16 o_acc[NDT];
#pragma unroll
  for (int t = 0; t < NDT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o_acc[t][r] = 0.f;
  f32x16 s_acc;
  u32x4 pq[2];                                     // P^T of the current tile: one operand per 16 keys
  float mc_run = -__builtin_inff(), l_run = 0.f;

  // Operand fragments are requested one product ahead: V's before the softmax or right behind the barrier,
  // K's between the MFMAs of the first product (left to itself the compiler reads one fragment, waits
  // for it and multiplies: 2.5 times as long per tile).
  V8 kf[NKK], vf[2][NDT];
  auto read_k = [&](int slot, int kk) __attribute__((always_inline)) {
    kf[kk] = __builtin_bit_cast(V8, *(const MLT_LDS u32x4*)(uintptr_t)(grp0 + slot * L::TILE_B + (uint32_t)(k_frag ^ (kk << 5))));
  };
  auto read_v = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        const uint32_t a = grp0 + slot * L::TILE_B + (uint32_t)(v_frag ^ (dt << 6)) + g * 16 * ROWB;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLT_LDS s16x4*)(uintptr_t)a);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((MLT_LDS s16x4*)(uintptr_t)(a + 8 * ROWB));
        vf[g][dt] = join_tr<V8>(lo, hi);
      }
  };
  // S^T = K Q^T
  auto scores = [&]() __attribute__((always_inline)) {
    f32x16 z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    s_acc = mfma32(kf[0], qf[0], z);
#pragma unroll
    for (int kk = 1; kk < NKK; ++kk) s_acc = mfma32(kf[kk], qf[kk], s_acc);
  };
  // O^T += V^T P^T, and the K fragments from ring slot `slot` (on a wavefront's last tile nobody uses them)
  auto outputs = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt) {
        o_acc[dt] = mfma32(vf[g][dt], __builtin_bit_cast(V8, pq[g]), o_acc[dt]);
        __builtin_amdgcn_sched_barrier(0);
        read_k(slot, g * NDT + dt);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  static_assert(2 * NDT == NKK, "one K fragment per MFMA");
  // softmax of S_t (in s_acc) -> pq, mc_run, rescaled o_acc and l_run; the lazy rescale of mha_pp_kernel.
  // A row may have seen no key at all yet (its keys are with other groups, or masked): its maximum is
  // then -inf and the weights are taken against 0, which makes them exp2(-inf) = 0.
  auto softmax = [&](int t) __attribute__((always_inline)) {
    if (t >= t_mask) {
      const int limit = CAUSAL && my_q < Sk - 1 ? my_q : Sk - 1;      // last visible key
      const int rel = limit - ((tb + kg + t * KW) * L::KEYS + 4 * h);
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (8 * (r >> 2) + (r & 3) > rel) s_acc[r] = -__builtin_inff();
    }
    float mx = s_acc[0];
#pragma unroll
    for (int r = 1; r < 15; r += 2) mx = max3(mx, s_acc[r], s_acc[r + 1]);
    mx = __builtin_fmaxf(mx, s_acc[15]);
    mx = both_halves_max(mx);
    const float top = mx * c;
    const bool grow = top - mc_run > PA_LAZY_T;
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
      const float alpha = grow ? __builtin_amdgcn_exp2f(mc_run - top) : 1.f;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o_acc[dt][r] *= alpha;
      mc_run = grow ? top : mc_run;
    }
    const float ref = mc_run == -__builtin_inff() ? 0.f : mc_run;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_acc[r], c, -ref));
      const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s_acc[r + 1], c, -ref));
      pq[r / 8][(r / 2) & 3] = Elem<Tag>::pack2(p0, p1);
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) asm volatile("" : "+v"(pq[g]));   // (not to sink below the next barrier)
  };
  auto sync = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    MLT_BARRIER();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
  };

  // Tiles that must have landed when interval t begins: s_0 .. s_{2t+2}; up to R - 4 tiles behind those stay
  // in flight as long as they all exist (the last of this group's K tiles is s_{2 Tg - 3}).
  auto wait_tiles = [&](int t) __attribute__((always_inline)) {
    if (2 * t + R - 2 <= 2 * Tg - 3) __builtin_amdgcn_s_waitcnt(wait_imm((R - 4) * L::LPW, 15));
    else __builtin_amdgcn_s_waitcnt(wait_imm(0, 15));
  };
  // s_i: K_{(i+1)/2} for odd i, V_{i/2-1} for even i; interval t issues s_{2t+R-1} and s_{2t+R}, one of each
  constexpr bool K_FIRST = R % 2 == 0;
  constexpr int TK = K_FIRST ? R / 2 : (R + 1) / 2, TV = K_FIRST ? R / 2 - 1 : (R - 1) / 2 - 1;   // of which step, at t = 0
  issue(0, Kh, voff_k, 0);
#pragma unroll
  for (int i = 1; i < R - 1; ++i) {
    if (i & 1) issue((i + 1) / 2, Kh, voff_k, i);
    else issue(i / 2 - 1, Vh, voff_v, i);
  }
  wait_tiles(0);
  sync();
  if (Tw > 0) {
#pragma unroll
    for (int kk = 0; kk < NKK; ++kk) read_k(0, kk);
    scores();
    if (!late) softmax(0);
  }
  sync();                                          // everyone is done with K_0
  int sk = 1;                                      // slot of s_{2t+1}; s_{2t+R-1} goes two slots before it, s_{2t+R} one before
  // interval t of a wavefront with work in steps t and t + 1 (CUR, NEXT)
  auto interval = [&](int t, auto CUR, auto NEXT) __attribute__((always_inline)) {
    const int sv = sk + 1 == R ? 0 : sk + 1;
    const int f2 = sk >= 1 ? sk - 1 : R - 1, f1 = f2 >= 1 ? f2 - 1 : R - 1;
    if (K_FIRST) issue(t + TK, Kh, voff_k, f1);
    else issue(t + TV, Vh, voff_v, f1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (CUR.value) {
      read_v(sv);
      __builtin_amdgcn_sched_barrier(0);
      if (late) softmax(t);
      __builtin_amdgcn_sched_barrier(0);
      outputs(sk);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (K_FIRST) issue(t + TV, Vh, voff_v, f2);
    else issue(t + TK, Kh, voff_k, f2);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NEXT.value) scores();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (CUR.value) {
      // the sum of the ROUNDED weights (what P V used), while the matrix pipe drains
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) l_run = Elem<Tag>::add_pair(pq[g][e], l_run);
      asm volatile("" : "+v"(l_run));
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (NEXT.value)
      if (!late) softmax(t + 1);
    wait_tiles(t + 1);
    sync();
    sk = sk + 2 >= R ? sk + 2 - R : sk + 2;
  };
  int t = 0;
  for (; t < Tw - 1; ++t) interval(t, std::true_type{}, std::true_type{});
  if (t < Tw) { interval(t, std::true_type{}, std::false_type{}); ++t; }
  for (; t < T; ++t) interval(t, std::false_type{}, std::false_type{});

  // ---- the key groups' results meet: outputs (fp32, unscaled) over the ring, maxima and sums behind it
  const float l_tot = both_halves_sum(l_run);
  float* stat = reinterpret_cast<float*>(smem + L::STAT_OFF);
  if (h == 0) {
    stat[(wave * 32 + lq) * 2] = mc_run;
    stat[(wave * 32 + lq) * 2 + 1] = l_tot;
  }
  // register quad g of tile t holds d = 32 t + 8 g + 4 h .. +3 of row lq
  float* park = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int t = 0; t < NDT; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4_mem*>(park + (wave * 32 + lq) * L::PSTR + 32 * t + 8 * g + 4 * h) =
          f32x4{o_acc[t][4 * g], o_acc[t][4 * g + 1], o_acc[t][4 * g + 2], o_acc[t][4 * g + 3]};
  __syncthreads();
#pragma unroll
  for (int i = 0; i < L::BM * L::CPR / 512; ++i) {
    const int e = tid + i * 512, r = e / L::CPR, d = (e % L::CPR) * 8;
    const int gq = qt * L::BM + r;
    if (gq >= Sq) continue;
    float m[KW], w[KW], M = -__builtin_inff(), sum = 0.f;
#pragma unroll
    for (int g = 0; g < KW; ++g) {
      m[g] = stat[((g * QW + r / 32) * 32 + r % 32) * 2];
      M = __builtin_fmaxf(M, m[g]);
    }
    const float ref = M == -__builtin_inff() ? 0.f : M;
    f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < KW; ++g) {
      const int row = (g * QW + r / 32) * 32 + r % 32;
      w[g] = __builtin_amdgcn_exp2f(m[g] - ref);
      sum += stat[row * 2 + 1] * w[g];
      const f32x4 a = *reinterpret_cast<const f32x4_mem*>(park + row * L::PSTR + d);
      const f32x4 b = *reinterpret_cast<const f32x4_mem*>(park + row * L::PSTR + d + 4);
#pragma unroll
      for (int x = 0; x < 4; ++x) { lo[x] += a[x] * w[g]; hi[x] += b[x] * w[g]; }
    }
    const int64_t row = (int64_t)bh * Sq + gq;
    if (SPLIT) {
      const int64_t prow = (int64_t)blockIdx.y * (total / nq) * Sq + row;
      if (d == 0) { ps[prow * 2] = M; ps[prow * 2 + 1] = sum; }
      *reinterpret_cast<f32x4_mem*>(po + prow * D + d) = lo;
      *reinterpret_cast<f32x4_mem*>(po + prow * D + d + 4) = hi;
    } else {
      const float inv = 1.f / sum;
      // (plain, unlike mha_pp.hip: these kernels' results are small, and the next call finds them in a cache. Call alone / with the copy to
      // B x S x H x D behind it, us, plain and non-temporal: 1 x 16 x 1024 x 64 causal 11.05 / 15.9 and 11.0 / 16.3, 1 x 16 x 2048 x 128 causal 33.5 /
      // 42.2 and 32.8 / 42.5, 8 x 16 x 256 x 64 8.23 / 13.65 and 8.13 / 13.8)
      *reinterpret_cast<u32x4_mem*>(O + row * D + d) =
          u32x4{Elem<Tag>::pack2(lo[0] * inv, lo[1] * inv), Elem<Tag>::pack2(lo[2] * inv, lo[3] * inv),
                Elem<Tag>::pack2(hi[0] * inv, hi[1] * inv), Elem<Tag>::pack2(hi[2] * inv, hi[3] * inv)};
    }
  }
}

// The ranges' partial results of a row, in index order: a lane owns 8 output columns. `rows` counts all
// batch * heads * Sq rows.
template <typename Tag, int D>
__global__ __launch_bounds__(256) void mha_ks_merge_kernel(const float* __restrict__ po, const float* __restrict__ ps,
                                                           uint16_t* __restrict__ O, int64_t rows, int nsplit) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t row = e / (D / 8);
  const int d = (int)(e % (D / 8)) * 8;
  if (row >= rows) return;
  float M = -__builtin_inff();
  for (int s = 0; s < nsplit; ++s) M = __builtin_fmaxf(M, ps[(s * rows + row) * 2]);
  const float ref = M == -__builtin_inff() ? 0.f : M;
  float sum = 0.f;
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < nsplit; ++s) {
    const int64_t prow = s * rows + row;
    const float w = __builtin_amdgcn_exp2f(ps[prow * 2] - ref);
    sum += ps[prow * 2 + 1] * w;
    const f32x4 a = *reinterpret_cast<const f32x4_mem*>(po + prow * D + d);
    const f32x4 b = *reinterpret_cast<const f32x4_mem*>(po + prow * D + d + 4);
#pragma unroll
    for (int x = 0; x < 4; ++x) { lo[x] += a[x] * w; hi[x] += b[x] * w; }
  }
  const float inv = 1.f / sum;
  *reinterpret_cast<u32x4_mem*>(O + row * D + d) =
      u32x4{Elem<Tag>::pack2(lo[0] * inv, lo[1] * inv), Elem<Tag>::pack2(lo[2] * inv, lo[3] * inv),
            Elem<Tag>::pack2(hi[0] * inv, hi[1] * inv), Elem<Tag>::pack2(hi[2] * inv, hi[3] * inv)};
}

template <typename Tag, int D, int QW, bool SPLIT, bool CAUSAL>
int launch_ks(const MhaArgs& a, int nsplit, float* scratch, hipStream_t s) {
  typedef KsCfg<D, QW> L;
  auto kern = mha_ks_kernel<Tag, D, QW, SPLIT, CAUSAL>;
  static thread_local int configured_dev = -1;          // opt in to > 64 KB LDS once per device
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MLT_ERR_DEVICE;
  if (configured_dev != dev) {
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, L::SMEM) != hipSuccess) {
      (void)hipGetLastError();
      return MLT_ERR_LAUNCH;
    }
    configured_dev = dev;
  }
  const int64_t nq = (a.Sq + L::BM - 1) / L::BM, total = a.B * a.H * nq, rows = a.B * a.H * a.Sq;
  if (total > 0x7fffffff) return MLT_ERR_UNSUPPORTED;
  float c = (a.scale < 0 ? -a.scale : a.scale) * 1.4426950408889634f;   // c > 0 always, as in launch_mha_pp
  if (c < 1e-30f) c = 1e-30f;
  float* ps = SPLIT ? scratch + (int64_t)nsplit * rows * D : nullptr;
  const int xcds = mha_xcd_word((int)total, CAUSAL, D, 32);
  hipLaunchKernelGGL(kern, dim3((unsigned)total, SPLIT ? nsplit : 1), dim3(512), L::SMEM, s, a.Q, a.K, a.V, a.O, scratch, ps,
                     (int)a.Sq, (int)a.Sk, (int)nq, (int)total,
                     xcds, c, a.scale < 0 ? 1 : 0, masked_map((int)total, (int)nq, (int)a.Sq, L::BM, CAUSAL, D, xcds));
  if (hipGetLastError() != hipSuccess) return MLT_ERR_LAUNCH;
  if (!SPLIT) return MLT_OK;
  hipLaunchKernelGGL((mha_ks_merge_kernel<Tag, D>), dim3((unsigned)((rows * (D / 8) + 255) / 256)), dim3(256), 0, s,
                     scratch, ps, a.O, rows, nsplit);
  return hipGetLastError() == hipSuccess ? MLT_OK : MLT_ERR_LAUNCH;
}

template <typename Tag, int D, int QW>
int run_ks_q(const MhaArgs& a, int nsplit, float* scratch, hipStream_t s) {
  if (a.causal) return nsplit > 1 ? launch_ks<Tag, D, QW, true, true>(a, nsplit, scratch, s) : launch_ks<Tag, D, QW, false, true>(a, 1, nullptr, s);
  return nsplit > 1 ? launch_ks<Tag, D, QW, true, false>(a, nsplit, scratch, s) : launch_ks<Tag, D, QW, false, false>(a, 1, nullptr, s);
}

template <typename Tag, int D>
int run_ks_t(const MhaArgs& a, int bm, int nsplit, float* scratch, hipStream_t s) {
  if (bm == 64) return run_ks_q<Tag, D, 2>(a, nsplit, scratch, s);
  return run_ks_q<Tag, D, 4>(a, nsplit, scratch, s);
}

}  // namespace

int run_mha_ks(const MhaArgs& a, int bm, int nsplit, float* scratch, hipStream_t s) {
  if (a.dtype == MLT_BF16)
    return a.D == 128 ? run_ks_t<bf16_tag, 128>(a, bm, nsplit, scratch, s) : run_ks_t<bf16_tag, 64>(a, bm, nsplit, scratch, s);
  return a.D == 128 ? run_ks_t<f16_tag, 128>(a, bm, nsplit, scratch, s) : run_ks_t<f16_tag, 64>(a, bm, nsplit, scratch, s);
}

}  // namespace mlt
