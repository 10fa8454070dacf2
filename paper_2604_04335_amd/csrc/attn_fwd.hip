// DiT denoising-step self-attention forward for gfx950 (MI355X): the 128-row and the ping-pong kernel, and the launch
// interface.  The tile code they share (and its description) is in attn_device.h.
#include "attn_device.h"

namespace dit {

// ---------------------------------------------------------------------------------------------
// Kernel A: 4 wavefronts, 128 query rows per workgroup.  The workgroups of a compute unit do not synchronise.
//
// A wavefront works one tile ahead (tile_step): the scores of tile t+1 are contracted while tile t goes through its
// exponentials and into O^T, so that its matrix and vector instructions overlap inside one instruction stream.  With the
// three back to back the two pipes of a SIMD took turns unless another wavefront happened to be at the right place: a
// wavefront alone on its SIMD used each of them a third of the time.  Alone it is bound by its own instruction issue (about
// five cycles each, 195 instructions a tile at head dimension 64), which is why the main loop has neither address
// arithmetic (slots of the K / V rings are immediate offsets, the loads run on pointers) nor tests.  MI355X, us, the kernel
// with the three back to back / this one: 1024 rows x 8 heads, D 64 15.7 / 11.7;  16384 x 1, D 64 199 / 133;  410 x 24, D 64
// 8.7 / 7.5;  image batch, D 64 (410 to 4250 rows x 24) 349 / 327;  9000 x 24, D 64 545 / 497;  1024 x 8, D 128 22.1 / 17.0;
// 4951 x 3, D 128 88.7 / 60.6;  3600 x 24, D 128 170 / 154.  (Slower: cross-attention at D 64 in two rounds of six to eight
// tiles, 7912 x 24 against 357 keys 30.2 / 31.8, 400 keys 32.2 to 33.7 / 33.9 to 35.4, 500 keys 36.8 to 38.8 / 37.9 to 39.5.)
//
// Two K and V ring slots let several workgroups share a compute unit: three at head dimension 64, two at 128 (a third
// wavefront per SIMD at 64, in 159 registers, fills more of the issue slots: image batch 344 with two, 332 with three).
// A step's direct loads stand behind its first MFMAs, one each (every second one at 128): issued in a burst behind the
// barrier, the wavefronts wait for one another on the compute unit's path to memory.  us, burst / spread: 3600 x 24, D 128
// 161 / 149, 46618 x 24 against 512 keys 323 / 318, 16384 x 1, D 64 136.8 / 134.7, image batch 328 / 326.
// Four slots are for workgroups that have a compute unit to themselves (head dimension 128; see launch_p): a barrier every
// second tile.
// ---------------------------------------------------------------------------------------------
template <int D>
constexpr int kWgsPerCu128 = D == 64 ? 3 : 2;

template <class T>
constexpr int kWavesPerSimd = T::NBUF > 2 ? 2 : kWgsPerCu128<T::D>;

template <class T, class P>
__global__ void __attribute__((amdgpu_flat_work_group_size(T::NT, T::NT), amdgpu_waves_per_eu(kWavesPerSimd<T>, kWavesPerSimd<T>)))
attn_fwd_kernel(const WorkItem* items, P p) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass needs the kernel's name only, and fails on the second instance of a body
  extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
  lds_char* smem = (lds_char*)smem_generic;
  lds_slot* s_item = reinterpret_cast<lds_slot*>(smem + T::ITEM_OFF);

  constexpr int NB = T::NBUF;
  const LaunchClock clock0 = launch_clock_begin(p);
  const int tid = threadIdx.x;
  const int64_t row_stride_b = (int64_t)p.n_heads * T::D * 2;
  const float c = p.c_log2;
  // Per-lane constants are recomputed where an item starts or ends; kept live through the tile loop they are spilled.
  auto fresh_lane = [&]() {
    int t = tid;
    asm volatile("" : "+v"(t));
    Lane<T> l;
    l.init(t, row_stride_b);
    return l;
  };
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t kvoff[T::LPT], vvoff[T::LPT];  // lane offsets of the load instructions of a whole tile
  {
    const Lane<T> L0 = fresh_lane();
#pragma unroll
    for (int i = 0; i < T::LPT; ++i) {
      kvoff[i] = L0.kvoff + (uint32_t)(i * T::GROUP) * (uint32_t)row_stride_b;
      vvoff[i] = L0.vvoff + (uint32_t)(i * T::GROUP) * (uint32_t)row_stride_b;
    }
  }
  const uint32_t lds_wave = (uint32_t)(uintptr_t)smem + (uint32_t)wave * 1024u;
  const int64_t tile_stride_b = (int64_t)T::BN * row_stride_b;

  // The index of the next item is requested towards the end of an item, into the slot of the other parity; a barrier
  // between that write and the end of the item makes it visible to every wave before it is read.
  const bool one_round = single_round(p);
  uint32_t item_idx = blockIdx.x;
  int par = 0;

  while (item_idx < p.n_items) {
    par ^= 1;  // the next index goes to s_item[par], see below
    const ItemCtx<T> X = begin_item<T, P>(p, items, fresh_lane(), item_idx, row_stride_b);
    const int kv_len = X.it.kv_len, nt = X.nt;

    // Tile ti, which starts at base, -> its ring slot.  Only for sequences of two tiles or more, whose tiles are all loaded
    // whole, the last one as the last BN keys.
    const int64_t last_b = (int64_t)(kv_len - T::BN) * row_stride_b;
    const char *const klast = X.kbase + last_b, *const vlast = X.vbase + last_b;
    auto load_k = [&](int ti, const char* base) {
      const uint32_t dst = lds_wave + T::K_OFF + (uint32_t)(ti & (NB - 1)) * T::TILE_B;
#pragma unroll
      for (int i = 0; i < T::LPT; ++i) lds_dma_16(base, kvoff[i], dst + i * T::NWAVES * 1024);
    };
    auto load_v = [&](int ti, const char* base) {
      const uint32_t dst = lds_wave + T::V_OFF + (uint32_t)(ti & (NB - 1)) * T::TILE_B;
#pragma unroll
      for (int i = 0; i < T::LPT; ++i) lds_dma_16(base, vvoff[i], dst + i * T::NWAVES * 1024);
    };
    // Q goes through slots that the first tiles do not need yet: two wavefronts' rows in K slot 1, two in V slot 1.  As
    // register loads (256 cache-line requests a wavefront instead of 64) the first loads of an item of 512 keys took 3 100
    // cycles of 31 000 to issue.  us: 1024 x 8, D 128 18.2 / 17.6, D 64 12.57 / 12.43;  46618 x 24 against 512 keys, D 128
    // 342 / 336, 226 keys 221 / 214.  (In the ping-pong kernel, whose buffers are all busy then, not worth a buffer.)
    constexpr int PER = T::TILE_B / (32 * T::ROW_B);  // wavefronts per slot
    static_assert(T::NWAVES == 2 * PER, "rows of four wavefronts in two slots");
    const uint32_t spare = (uint32_t)(uintptr_t)smem + (wave < PER ? T::K_OFF : T::V_OFF) + T::TILE_B + (uint32_t)(wave % PER) * (32 * T::ROW_B);
    {
      const Lane<T> L = fresh_lane();
      q_rows_load<T>(p, L, X.it, row_stride_b, X.head_off, spare);
      tile_load_one<T>(X.kbase, row_stride_b, 0, kv_len, L.lrow, L.kcol, kvoff[0], smem, T::K_OFF, wave);
      tile_load_one<T>(X.vbase, row_stride_b, 0, kv_len, L.lrow, L.vcol, vvoff[0], smem, T::V_OFF, wave);
    }

    f32x16 o[T::NDB];
#pragma unroll
    for (int db = 0; db < T::NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    float m_ref = -1.0e30f;  // finite: (m_ref - m) * c stays finite
    float l_run = 0.f, mx = 0.f;
    f32x16 sa[T::NKB], sb[T::NKB];
    uint32_t pb[T::NKB][8];
    int ka[T::NKS], va[T::NDB];
    fresh_lane().operand_addrs((uint32_t)(uintptr_t)smem, (uint32_t)(uintptr_t)smem, ka, va);

    if (nt == 1 && tid == 0 && !one_round) s_item[par] = take_item(p);  // visible after the barrier below
    if (nt > 1)
      wait_loads_but<T::LPT>();  // V(0) is awaited with K(1), before step 0
    else
      wait_loads();
    bf16x8 qf[T::NKS];
    q_rows_read<T>(p, fresh_lane(), spare, qf);
    wg_barrier();
    if (nt > 1) load_k(1, nt == 2 ? klast : X.kbase + tile_stride_b);
    if (NB > 2 && nt > 2) load_k(2, nt == 3 ? klast : X.kbase + 2 * tile_stride_b);
    if (NB > 2 && nt > 1) load_v(1, nt == 2 ? vlast : X.vbase + tile_stride_b);
    mfma_stream<T, false, 0, T::NQK, kPrefetch>(smem, va, ka, pb, qf, o, sa);
    scores_ready<T>(sa);
    if (nt > 1) mx = tile_max<T>(sa);
    // Step t: S(t) is in sc; leaves S(t+1) in sn.  Every PER_BAR steps there is a barrier, behind which K(t+1) and V(t) (with
    // two steps to a barrier also K(t+2) and V(t+1)) have landed for everyone and nobody reads the tiles before them any
    // more: their slots take the tiles behind them.  A step of the main loop (MAIN) loads tiles that are not a sequence's
    // last, from running pointers.
    constexpr int PER_BAR = NB / 2;
    const char* kp = X.kbase + (PER_BAR + 1) * tile_stride_b;
    const char* vp = X.vbase + PER_BAR * tile_stride_b;
    constexpr int NLOAD = 2 * PER_BAR * T::LPT, EVERY = T::EVERY;
    static_assert(EVERY * NLOAD <= T::NQK + T::NPV, "a step's loads fit its slots");
    auto step = [&](auto uc, auto mainc, f32x16(&sc)[T::NKB], f32x16(&sn)[T::NKB], int t) {
      constexpr int U = decltype(uc)::value;  // t % UNROLL in the main loop, t % 2 behind it
      constexpr bool MAIN = decltype(mainc)::value;
      constexpr bool BAR = U % PER_BAR == 0;
      if constexpr (BAR) {
        wait_loads();
        wg_barrier();
      }
      const bool ask = !MAIN && t + 2 == nt && tid == 0 && !one_round;
      uint32_t next_item = 0;
      auto load_i = [&](auto jc) {
        constexpr int j = decltype(jc)::value, i = j % T::LPT, n = j / (2 * T::LPT);
        if constexpr (j / T::LPT % 2 == 0)
          lds_dma_16_at<T::K_OFF + (U + PER_BAR + 1 + n) % NB * T::TILE_B + i * T::NWAVES * 1024>(kp + n * tile_stride_b, kvoff[i], lds_wave);
        else
          lds_dma_16_at<T::V_OFF + (U + PER_BAR + n) % NB * T::TILE_B + i * T::NWAVES * 1024>(vp + n * tile_stride_b, vvoff[i], lds_wave);
      };
      if constexpr (!MAIN) {
        if (ask) next_item = take_item(p);
        if constexpr (BAR) {
#pragma unroll
          for (int n = 0; n < PER_BAR; ++n) {
            const int tk = t + PER_BAR + 1 + n, tv = t + PER_BAR + n;
            if (tk < nt) load_k(tk, tk == nt - 1 ? klast : kp + n * tile_stride_b);
            if (tv < nt) load_v(tv, tv == nt - 1 ? vlast : vp + n * tile_stride_b);
          }
        }
      } else if constexpr (BAR && EVERY == 0) {
        static_for<0, NLOAD>(load_i);
      }
      raise_reference<T>(mx, c, o, m_ref, l_run);
      const float mc = m_ref * c;
      tile_step<T, MAIN ? (U + 1) % NB * T::TILE_B : 0, MAIN ? U % NB * T::TILE_B : 0, kPrefetch>(
          va, ka, pb, qf, o, sc, sn, c, mc, mx, [&](auto jc) {
            constexpr int J = decltype(jc)::value;
            if constexpr (MAIN && BAR && EVERY != 0) {
              if constexpr (J % EVERY == EVERY / 2 && J / EVERY < NLOAD) load_i(IC<J / EVERY>{});
            }
          });
      if constexpr (BAR) {
        kp += PER_BAR * tile_stride_b;
        vp += PER_BAR * tile_stride_b;
      }
      if constexpr (!MAIN) {
#pragma unroll
        for (int ks = 0; ks < T::NKS; ++ks) ka[ks] ^= (((t + 1) ^ (t + 2)) & (NB - 1)) * T::TILE_B;
#pragma unroll
        for (int db = 0; db < T::NDB; ++db) va[db] ^= ((t ^ (t + 1)) & (NB - 1)) * T::TILE_B;
      }
      l_run += row_sum<T>(pb);
      asm volatile("" : "+v"(l_run));
      if (ask) s_item[par] = next_item;
    };
    static_assert(NB == 2 || NB == 4, "slots by exclusive or; the parity of the scores follows t");
    constexpr int UNROLL = NB;
    int t = 0;
    for (; t + UNROLL + PER_BAR + 1 < nt; t += UNROLL)
      static_for<0, UNROLL / 2>([&](auto ic) {
        constexpr int I = 2 * decltype(ic)::value;
        step(IC<I>{}, IC<1>{}, sa, sb, t + I);
        step(IC<I + 1>{}, IC<1>{}, sb, sa, t + I + 1);
      });
    // The last steps: t is a multiple of NB here; the addresses follow the slots.
#pragma unroll
    for (int ks = 0; ks < T::NKS; ++ks) ka[ks] ^= T::TILE_B;
    for (; t + 2 < nt; t += 2) {
      step(IC<0>{}, IC<0>{}, sa, sb, t);
      step(IC<1>{}, IC<0>{}, sb, sa, t + 1);
    }
    if (t + 1 < nt) {
      step(IC<0>{}, IC<0>{}, sa, sb, t);
#pragma unroll
      for (int kb = 0; kb < T::NKB; ++kb) sa[kb] = sb[kb];
    }
    if (nt > 1) {
      wait_loads();
      wg_barrier();
    }
    const Lane<T> L = fresh_lane();
    tile_softmax<T, true>(sa, L.hh, tail_rows<T>(kv_len), c, pb, o, m_ref, l_run);
    mfma_stream<T, true, 0, 0, kPrefetch>(smem, va, ka, pb, qf, o, sa);
    l_run += row_sum<T>(pb);

    // The rows are staged in the K ring, which nobody reads or loads into behind the barrier of the last tile, or, with one
    // tile and no such barrier, where Q was.
    int qrow = L.wave * 32 + L.l32;
    const bool row_valid = qrow < X.it.q_rows;
    if (!row_valid) qrow = X.it.q_rows - 1;
    const uint32_t stage = nt > 1 ? (uint32_t)(uintptr_t)smem + T::K_OFF + (uint32_t)wave * (32 * T::ROW_B) : spare;
    store_out<T>(p, L, X.it, row_stride_b, X.head_off, qrow, row_valid, o, l_run, m_ref, stage);
    if (one_round) break;
    wg_barrier();  // the next item's first loads overwrite ring slot 0
    item_idx = __builtin_amdgcn_readfirstlane(s_item[par]);
  }
  launch_clock_end(p, clock0);
#endif
}

// ---------------------------------------------------------------------------------------------
// Kernel B (ping-pong): 8 wavefronts, 256 query rows per workgroup, one workgroup per compute unit.
//
// Wavefronts w and w+4 share a SIMD.  Group 0 (waves 0-3) and group 1 (waves 4-7) run the same program one phase
// apart, with a workgroup barrier after every phase: while one group keeps the matrix pipe busy, the other does its
// softmax on the vector ALU.  A phase works through a PAIR of consecutive 64-key tiles (a K / V buffer holds a pair):
// half as many barriers and MFMA-stream start-ups per key as one tile per phase, which was worth 14 % fewer cycles per
// key.  The softmax stays per tile (one reference decision per row and 64 keys, exactly as in the 128-row kernel), so
// both kernels produce the same bits; the second tile's rescale of O^T, which in a tile-by-tile pass happens after the
// first tile's PV MFMAs, is deferred into the matrix phase (pp_stream).  With P(t) the pair of tiles 2t, 2t+1, phase p
// of an item (p = 0 after the first barrier):
//     group 0:  QK(P0) at p=0,  softmax(Pt) at p=2t+1,  PV(Pt)+QK(Pt+1) at p=2t+2
//     group 1:  idle   at p=0,  QK(P0) at p=1, softmax(Pt) at p=2t+2, PV(Pt)+QK(Pt+1) at p=2t+3
// K(Pt+1) and V(Pt) are therefore read in phases 2t+2 and 2t+3 only; their buffers (parity of the pair index) can be
// refilled with K(Pt+3) / V(Pt+2) from phase 2t+4 on.  Loads are issued by wavefronts in their vector phase only (a
// wavefront in its matrix phase is the critical path and issues nothing but MFMAs and operand reads; a direct load
// holds its wavefront for ~64 cycles), each for its own rows and those of the wavefront four away, and the two groups
// share the issue: group 1 issues V(Pt+1) at the start of phase 2t+2 and awaits it at the end of phase 2t+3, before the
// barrier that lets group 0 read it; group 0 issues K(Pt+1) at the start of phase 2t+1 (its buffer was last read in
// phase 2t-1) and awaits it at the end of the same phase, behind its two softmaxes (about 0.8 us later: K comes from
// L2 or the memory-side cache, whose latency that covers).  All of it in group 1 made that group's vector phase the
// longest phase by ~500 cycles.  A sequence with an odd number of tiles ends in a pair of one tile; the QK MFMAs of the
// missing tile run on whatever its buffer half holds and their scores are never read.
// ---------------------------------------------------------------------------------------------
template <class T, class P>
__global__ void __attribute__((amdgpu_flat_work_group_size(T::NT, T::NT), amdgpu_waves_per_eu(2, 2)))
attn_fwd_pp_kernel(const WorkItem* items, P p) {
#if defined(__HIP_DEVICE_COMPILE__)  // the host pass needs the kernel's name only, and fails on the second instance of a body
  static_assert(T::NWAVES == 8 && T::SUBS == 2, "two groups of four wavefronts, two tiles per phase");
  extern __shared__ __attribute__((aligned(1024))) char smem_generic[];
  lds_char* smem = (lds_char*)smem_generic;
  lds_slot* s_item = reinterpret_cast<lds_slot*>(smem + T::ITEM_OFF);

  const LaunchClock clock0 = launch_clock_begin(p);
  const int tid = threadIdx.x;
  const int64_t row_stride_b = (int64_t)p.n_heads * T::D * 2;
  const float c = p.c_log2;
  // Per-lane constants.  Only the two load offsets stay in registers for the life of the kernel; everything else is
  // recomputed where an item starts or ends (fresh_lane: some twenty instructions), from a thread index that the
  // compiler cannot see through.  Kept live instead, they sit in registers that the pair loop needs and are spilled
  // around it: sixty scratch instructions per wavefront and item, on the one vector-memory path that the item's first
  // loads and output stores also go through.
  auto fresh_lane = [&]() {
    int t = tid;
    asm volatile("" : "+v"(t));
    Lane<T> l;
    l.init(t, row_stride_b);
    return l;
  };
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave >> 2;
  uint32_t kvoff, vvoff;
  {
    const Lane<T> L0 = fresh_lane();
    kvoff = L0.kvoff;
    vvoff = L0.vvoff;
  }

  // The index of the next item is requested towards the end of an item, into the slot of the other parity; a barrier
  // between that write and the end of the item makes it visible to every wave before it is read.
  const bool one_round = single_round(p);
  uint32_t item_idx = blockIdx.x;
  int par = 0;

  while (item_idx < p.n_items) {
    par ^= 1;  // the next index goes to s_item[par], see below
    const ItemCtx<T> X = begin_item<T, P>(p, items, fresh_lane(), item_idx, row_stride_b);
    const int kv_len = X.it.kv_len, nt = X.nt;  // nt: 64-key tiles
    const int npairs = (nt + 1) >> 1;

    // Tile ti of K / V -> half ti&1 of the buffer of parity (ti>>1)&1, for the rows of wavefront `wave`.
    // dw: 0 for this wavefront's own rows, `other` for those of the wavefront four away
    auto load_k = [&](int ti, const Lane<T>& L, int dw) {
      if (ti < nt)
        tile_load_one<T>(X.kbase, row_stride_b, tile_first_key<T>(ti, kv_len), kv_len, L.lrow + dw * T::RPI, L.kcol,
                         kvoff + (uint32_t)(dw * T::RPI) * (uint32_t)row_stride_b, smem,
                         T::K_OFF + ((ti >> 1) & 1) * T::BUF_B + (ti & 1) * T::TILE_B, wave + dw);
    };
    auto load_v = [&](int ti, const Lane<T>& L, int dw) {
      if (ti < nt)
        tile_load_one<T>(X.vbase, row_stride_b, tile_first_key<T>(ti, kv_len), kv_len, L.lrow + dw * T::RPI, L.vcol,
                         vvoff + (uint32_t)(dw * T::RPI) * (uint32_t)row_stride_b, smem,
                         T::V_OFF + ((ti >> 1) & 1) * T::BUF_B + (ti & 1) * T::TILE_B, wave + dw);
    };
    // Inside the pair loop the group that is in its vector phase issues loads for both groups (its own rows and those
    // of the wavefront four away).  While the tiles are whole interior tiles (every tile but the last of a sequence)
    // their rows form one run of 2 * LPT load rounds, GROUP rows apart: the addresses come from one running pointer
    // and the load issue, which sits on the critical path of the vector phase, carries no per-tile tests or
    // multiplications.
    const int other = group == 1 ? -4 : 4;  // the wavefront whose rows this one also loads
    const uint32_t d4 = (uint32_t)(other * T::RPI) * (uint32_t)row_stride_b;
    const int64_t round_b = (int64_t)T::GROUP * row_stride_b;
    auto load_k_pair_all = [&](int tp) {  // K tiles 2tp, 2tp+1 -> K buffer tp&1
      if (2 * tp + 1 < nt - 1) {
        const char* kp = X.kbase + (int64_t)(2 * tp) * T::BN * row_stride_b;
        const uint32_t lk = (uint32_t)(uintptr_t)smem + T::K_OFF + (tp & 1) * T::BUF_B + (uint32_t)wave * 1024u;
#pragma unroll
        for (int j = 0; j < 2 * T::LPT; ++j) {
          lds_dma_16(kp + j * round_b, kvoff, lk + j * T::NWAVES * 1024);
          lds_dma_16(kp + j * round_b, kvoff + d4, lk + j * T::NWAVES * 1024 + other * 1024);
        }
      } else {
        const Lane<T> L = fresh_lane();
        load_k(2 * tp, L, 0);
        load_k(2 * tp + 1, L, 0);
        load_k(2 * tp, L, other);
        load_k(2 * tp + 1, L, other);
      }
    };
    auto load_v_pair_all = [&](int tp) {  // V tiles 2tp, 2tp+1 -> V buffer tp&1
      if (2 * tp + 1 < nt - 1) {
        const char* vp = X.vbase + (int64_t)(2 * tp) * T::BN * row_stride_b;
        const uint32_t lv = (uint32_t)(uintptr_t)smem + T::V_OFF + (tp & 1) * T::BUF_B + (uint32_t)wave * 1024u;
#pragma unroll
        for (int j = 0; j < 2 * T::LPT; ++j) {
          lds_dma_16(vp + j * round_b, vvoff, lv + j * T::NWAVES * 1024);
          lds_dma_16(vp + j * round_b, vvoff + d4, lv + j * T::NWAVES * 1024 + other * 1024);
        }
      } else {
        const Lane<T> L = fresh_lane();
        load_v(2 * tp, L, 0);
        load_v(2 * tp + 1, L, 0);
        load_v(2 * tp, L, other);
        load_v(2 * tp + 1, L, other);
      }
    };
    // A wavefront none of whose 32 query rows exists (the ragged last query tile of a sequence, a half-height item of
    // a pack's last round) takes its part in the loads and barriers of the item and computes nothing: its SIMD and the
    // power it would draw go to the wavefront it shares the SIMD with.  Wavefront 0 always has rows.
    if (wave * 32 >= X.it.q_rows) {
      if (group == 0) load_k_pair_all(0);
      wait_loads();
      wg_barrier();
      if (group == 1) {
        load_v_pair_all(0);
        wg_barrier();
        wait_loads();
      }
      wg_barrier();
      for (int t = 0; t + 1 < npairs; ++t) {
        if (group == 1) load_v_pair_all(t + 1);
        if (group == 0) load_k_pair_all(t + 1);
        if (group == 0) wait_loads();
        wg_barrier();
        if (group == 1) wait_loads();
        wg_barrier();
      }
      wg_barrier();
      wg_barrier();
      if (group == 0) wg_barrier();
      if (one_round) break;
      item_idx = __builtin_amdgcn_readfirstlane(s_item[par]);
      continue;
    }
    bf16x8 qf[T::NKS];
    {
      // Only what phase 0 needs, Q and K(P0): the loads of an item's start and the stores of its end go through the
      // compute unit's one path to L2 at some 30 bytes a cycle, and Q, three pairs of tiles and the output rows there
      // at once (224 KB) were 7 500 cycles of every item.  V(P0) and K(P1), first read in phase 2, follow in phases 0
      // and 1, when that path is idle.  Q first: its rows come from memory (no compute unit has read them before), K
      // and V mostly from L2.
      // K(P0) is loaded by group 0 for both groups: group 1, which comes out of the item before a phase later and
      // with its output stores just issued, is what the first barrier waits for.
      load_q<T>(p, fresh_lane(), X.it, row_stride_b, X.head_off, X.qrow, qf);
      if (group == 0) load_k_pair_all(0);
    }

    f32x16 o[T::NDB];
#pragma unroll
    for (int db = 0; db < T::NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    float m_ref = -1.0e30f;  // finite: (m_ref - m) * c stays finite
    float l_run = 0.f;
    f32x16 s[2][T::NKB];
    uint32_t pb[2][T::NKB][8];
    int ka[T::NKS], va[T::NDB];  // ka: K buffer the next QK reads; va: V buffer the next PV reads
    fresh_lane().operand_addrs((uint32_t)(uintptr_t)smem, (uint32_t)(uintptr_t)smem, ka, va);
    float alpha1 = 1.f;
    uint64_t grown = 0;

    wait_loads();
    wg_barrier();  // Q and K(P0) of every wave have landed; phase 0 starts
    if (group == 1) {  // group 1 has no matrix work in phase 0: it requests V(P0), awaited behind its QK(P0)
      load_v_pair_all(0);
      wg_barrier();
    }
    pp_stream<T, 0, 2, kPrefetch>(va, ka, pb, qf, o, s, 0, 1.f);  // QK(P0)
#pragma unroll
    for (int ks = 0; ks < T::NKS; ++ks) ka[ks] ^= T::BUF_B;
    if (group == 1) wait_loads();
    wg_barrier();

    if (npairs == 1 && tid == 0 && !one_round) s_item[par] = take_item(p);  // two barriers follow in the last pair
    for (int t = 0; t + 1 < npairs; ++t) {
      // ---- vector phase: softmax of both tiles of pair t (whole tiles)
      // The next index is requested at the start of this phase and put into its slot at the end (visible after the
      // barriers of the last pair): the request takes about a microsecond, which thread 0's wavefront spends on its
      // softmaxes instead of waiting while seven wavefronts wait for it at the barrier.
      const bool ask = t + 2 == npairs && tid == 0 && !one_round;
      uint32_t next_item = 0;
      if (ask) next_item = take_item(p);
      if (group == 1) load_v_pair_all(t + 1);            // read from phase 2t+4 on
      if (group == 0) load_k_pair_all(t + 1);  // read from the next phase on
      tile_softmax<T, false>(s[0], 0, TailRows{0, T::BN}, c, pb[0], o, m_ref, l_run);  // no mask: hh unused
      grown = tile_softmax<T, false, true>(s[1], 0, TailRows{0, T::BN}, c, pb[1], o, m_ref, l_run, &alpha1);
      if (group == 0) wait_loads();
      if (ask) s_item[par] = next_item;
      wg_barrier();
      // ---- matrix phase: PV(Pt), QK(Pt+1)
      __builtin_amdgcn_s_setprio(1);
      pp_stream<T, 2, 2, kPrefetch>(va, ka, pb, qf, o, s, grown, alpha1);
      l_run = (l_run + row_sum<T>(pb[0])) * alpha1 + row_sum<T>(pb[1]);
      asm volatile("" : "+v"(l_run));  // the sums are taken here, not behind the barrier
      __builtin_amdgcn_s_setprio(0);
#pragma unroll
      for (int ks = 0; ks < T::NKS; ++ks) ka[ks] ^= T::BUF_B;
#pragma unroll
      for (int db = 0; db < T::NDB; ++db) va[db] ^= T::BUF_B;
      if (group == 1) wait_loads();  // pair t+1, issued at the start of this group's softmax(Pt)
      wg_barrier();
    }
    // ---- last pair: two tiles or one, the last of them masked; PV only
    if ((nt & 1) == 0) {
      tile_softmax<T, false>(s[0], 0, TailRows{0, T::BN}, c, pb[0], o, m_ref, l_run);
      grown = tile_softmax<T, true, true>(s[1], fresh_lane().hh, tail_rows<T>(kv_len), c, pb[1], o, m_ref, l_run, &alpha1);
      wg_barrier();
      __builtin_amdgcn_s_setprio(1);
      pp_stream<T, 2, 0, kPrefetch>(va, ka, pb, qf, o, s, grown, alpha1);
      l_run = (l_run + row_sum<T>(pb[0])) * alpha1 + row_sum<T>(pb[1]);
      asm volatile("" : "+v"(l_run));  // the sums are taken here, not behind the barrier
      __builtin_amdgcn_s_setprio(0);
    } else {
      tile_softmax<T, true>(s[0], fresh_lane().hh, tail_rows<T>(kv_len), c, pb[0], o, m_ref, l_run);
      wg_barrier();
      __builtin_amdgcn_s_setprio(1);
      pp_stream<T, 1, 0, kPrefetch>(va, ka, pb, qf, o, s, 0, 1.f);
      l_run += row_sum<T>(pb[0]);
      asm volatile("" : "+v"(l_run));
      __builtin_amdgcn_s_setprio(0);
    }
    wg_barrier();

    {
      const Lane<T> L = fresh_lane();
      int qrow = L.wave * 32 + L.l32;  // as in item_ctx
      const bool row_valid = qrow < X.it.q_rows;
      if (!row_valid) qrow = X.it.q_rows - 1;
      // Staging area of the rows.  Group 0 stores while group 1 runs its last matrix phase, which reads V only, and
      // every load of K has been awaited: it takes K buffer 0.  Group 1 stores while group 0 starts the next item and
      // loads its first tiles into both K buffers and V buffer 0: it takes V buffer 1, which is loaded into next by
      // group 1 itself, in the next item's pair loop behind two barriers.
      const uint32_t stage = (uint32_t)(uintptr_t)smem + (group == 0 ? T::K_OFF : T::V_OFF + T::BUF_B) +
                             (uint32_t)(wave & 3) * (32 * T::ROW_B);
      store_out<T>(p, L, X.it, row_stride_b, X.head_off, qrow, row_valid, o, l_run, m_ref, stage);
    }
    if (group == 0) wg_barrier();  // group 0 idles (after its stores) while group 1 runs its last matrix phase
    if (one_round) break;
    item_idx = __builtin_amdgcn_readfirstlane(s_item[par]);
  }
  launch_clock_end(p, clock0);
#endif
}

// The LDS limit of a kernel is set once per device (its first use there also loads the kernel's code).
template <class T, class P, void (*KERNEL)(const WorkItem*, P)>
static hipError_t prepare_t() {
  static bool attr_set[16] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 16 || !attr_set[dev]) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 16) attr_set[dev] = true;
  }
  return hipSuccess;
}

template <class T, class P, void (*KERNEL)(const WorkItem*, P)>
static hipError_t launch_t(const P& p, int grid, hipStream_t stream) {
  const hipError_t e = prepare_t<T, P, KERNEL>();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(KERNEL, dim3(grid), dim3(T::NT), T::LDS_BYTES, stream, p.items, p);
  return hipGetLastError();
}

using TilePP128 = Tile<128, 8, 64, 2>;
using TilePP64 = Tile<64, 8, 64, 2>;
using Tile128 = Tile<128, 4, 64, 1, 2, 2>;
using Tile128Burst = Tile<128, 4, 64>;
using Tile128Deep = Tile<128, 4, 64, 1, 4, 2>;
using Tile64 = Tile<64, 4, 64, 1, 2, 1>;

template <class P>
static hipError_t prepare_all() {
  hipError_t e = prepare_t<TilePP128, P, attn_fwd_pp_kernel<TilePP128, P>>();
  if (e == hipSuccess) e = prepare_t<TilePP64, P, attn_fwd_pp_kernel<TilePP64, P>>();
  if (e == hipSuccess) e = prepare_t<Tile128, P, attn_fwd_kernel<Tile128, P>>();
  if (e == hipSuccess) e = prepare_t<Tile128Burst, P, attn_fwd_kernel<Tile128Burst, P>>();
  if (e == hipSuccess) e = prepare_t<Tile128Deep, P, attn_fwd_kernel<Tile128Deep, P>>();
  if (e == hipSuccess) e = prepare_t<Tile64, P, attn_fwd_kernel<Tile64, P>>();
  return e;
}
hipError_t attn_fwd_prepare() {
  const hipError_t e = prepare_all<AttnParams>();
  return e == hipSuccess ? prepare_all<AttnListParams>() : e;
}

int attn_fwd_block_m(AttnKernel kernel) { return kernel == AttnKernel::kIndependent128 ? 128 : 256; }
int attn_fwd_wgs_per_cu(AttnKernel kernel, int head_dim) {
  if (kernel != AttnKernel::kIndependent128) return 1;
  return head_dim == 64 ? kWgsPerCu128<64> : kWgsPerCu128<128>;
}

AttnKernel attn_fwd_select(const int32_t* cu_seqlens, const int32_t* cu_seqlens_k, int32_t n_seqs, int32_t n_heads,
                           int head_dim, int n_cus) {
  // Measured on MI355X, us of the 128-row / the ping-pong kernel, rows x heads.
  const int32_t* ck = cu_seqlens_k ? cu_seqlens_k : cu_seqlens;
  int64_t rows = 0, items128 = 0, items256 = 0, tiles = 0, max_tiles = 0;  // tiles: key tiles of all 256-row items
  for (int32_t i = 0; i < n_seqs; ++i) {
    const int64_t lq = cu_seqlens[i + 1] - cu_seqlens[i], lk = ck[i + 1] - ck[i];
    if (lq == 0 || lk == 0) continue;
    const int64_t it = (lq + 255) / 256 * n_heads, nt = (lk + 63) / 64;
    rows += lq * n_heads;
    items128 += (lq + 127) / 128 * n_heads;
    items256 += it;
    tiles += it * nt;
    max_tiles = nt > max_tiles ? nt : max_tiles;
  }
  // Every 128-row item has a compute unit of its own: nothing is gained by longer ones.  D 128: 1280 x 24 25.7 / 30.9,
  // 2048 x 15 34.8 / 44.0, 2100 x 15 37.5 / 45.0, 4096 x 8 65.3 / 80, 1300 x 23 27.6 / 31.7, 16 of 200 x 8 8.4 / 11.8;  past it
  // 1300 x 24 35.8 / 32.1, 1408 x 24 37.1 / 32.5, 2048 x 17 50.3 / 44.3, 4096 x 9 94 / 81.  D 64: 1280 x 24 17.1 / 23.4, 410 x 24
  // 7.8 / 11.7;  past it 1300 x 24 23.4 / 24.6, 1792 x 24 30.6 / 30.4, 8192 x 6 121 / 120.
  if (items128 <= n_cus) return AttnKernel::kIndependent128;
  // Items with few key tiles (cross-attention against text keys): the 128-row kernel's workgroups have no idle phase at
  // the ends of an item.  46618 x 24, D 128: 77 keys 149 / 178, 226: 202 / 224, 512: 322 / 334, 640: 379 / 386 (8704 x 24: 73 /
  // 79), 768: 438 / 439;  D 64: 200 keys 112 / 148.  At D 64 one or two tiles are bound by Q and O, which the larger items move
  // better: 77 keys 109.3 / 102.9, 128 keys 109.0 / 95.7 (8704 x 24: 24.7 / 24.7 and 24.6 / 23.1).
  if (cu_seqlens_k != nullptr && tiles <= 5 * items256)
    return head_dim == 64 && tiles <= 2 * items256 ? AttnKernel::kPingPong256 : AttnKernel::kIndependent128;
  // The 256-row items take no longer than the longest of them: the ping-pong kernel's are the quicker ones.  D 128:
  // 1570 x 24 43.5 / 37.3, 410 and 2458 x 24 78.4 / 71.7, against 512 keys 19.6 / 18.3;  D 64: 1570 x 24 28.1 / 28.3, 2458 x 24
  // 45.2 / 44.3.
  if (tiles <= n_cus * max_tiles) return AttnKernel::kPingPong256;
  // Past one round at D 64 three workgroups of the 128-row kernel share a compute unit and are ahead: 512 x 24 heads x 18
  // sequences 45.4 / 51.6, 768 x 24 x 8 42.9 / 51.1, 1536 x 24 x 6 93 / 112, 3000 x 24 73 / 98, 4352 x 24 132 / 145, 6000 x 24 233 /
  // 287, 2458 x 24 x 4 164 / 174, 3000 x 12 x 7 203 / 213, 5120 x 24 x 2 331 / 336, 4352 x 24 x 4 451 / 509, 7000 x 24 318 / 337,
  // 8128 x 24 395 / 416, 9000 x 24 490 / 560, 20506 x 24 2450 / 2560, 46618 x 24 against 512 keys 172 / 205;  level at 1024 x 24 x
  // 8 (68.1 / 67.6), 512 x 24 x 16 (41.6 / 41.8), 10000 x 24 (639 / 641), 16384 x 16 (1078 / 1083) and 13000 x 10 x 2 (859 / 857).
  // Batches of several lengths: 3167, 537, 876 and 322 rows 85 / 104, 4 each of 4352, 2458, 1054 and 410 635 / 700, 410 to 4250
  // rows 325 / 350, 421 to 3916 rows x 12 86 / 89, 8192, 300 and 77 x 12 211 / 276.
  if (head_dim == 64) {
    // The exception: short items of self-attention that are two rounds for the ping-pong kernel and more than one for the
    // 128-row kernel, whose second round costs more than its share (a workgroup alone on its compute unit takes some 0.6 of
    // what three take together).  Its times scatter there, from card to card and with the rows: whole tiles 512 x 24 x 9 27.8 to
    // 30.2 / 26.5 to 28.6, 640 x 24 x 7 32.4 to 34.7 / 30.3 to 31.5, 768 x 8 x 20 38 to 42 / 35.6 to 38.4, 1024 x 24 x 5 47.2 to
    // 48.7 / 43.3 to 45.9, 1024 x 8 x 16 48.0 to 49.9 / 44.5 to 47.6;  ragged ones 410 x 24 x 9 23.5 to 28.9 / 24.4 to 26.2, 745 x 24
    // x 7 35.7 to 38.7 / 37.6 to 39.9, 925 x 12 x 10 40.9 to 42.8 / 39.7 to 44.1, 1054 x 24 x 4 43.7 to 45.2 / 42.6 to 47.3.  Up to 17
    // key tiles: 1152 x 24 x 4 45.5 / 45.5, 1200 x 24 x 4 49.4 / 49.9 to 52.9, 1280 x 24 x 4 51.3 / 52.4 to 55.2, 1536 x 24 x 3 55.0 /
    // 57.1 to 61.6.  Not where the 256-row items hold under 200 rows on average: 520 x 24 x 7 27.7 / 28.7, 588 x 24 x 7 29.8 / 30.4;
    // not with a third round: 1120 x 24 x 5 51.9 / 59.8, 1152 x 24 x 5 54.4 / 64.1;  not with one round: 300 x 24 x 10 14.8 / 20.4.
    const bool two_rounds = items128 > 3 * (int64_t)n_cus && items256 <= 2 * (int64_t)n_cus;
    if (cu_seqlens_k == nullptr && two_rounds && tiles <= 17 * items256 && rows >= 200 * items256) return AttnKernel::kPingPong256;
    return AttnKernel::kIndependent128;
  }
  // Else, at D 128, the ping-pong kernel (7 to 25 % ahead from 1.75 items per compute unit on: 4608 x 24 253 / 244, 5120 x 24 328 /
  // 279, 8000 x 16 515 / 425, 20506 x 6 1270 / 1062, 1024 x 24 x 8 118 / 106, 6000 and 3000 x 17 347 / 314), but for
  // cross-attention items of up to eleven key tiles (see above) and items that leave much of its last round empty.
  // (Comparisons of two kernels must be made on a warm chip: in the first ~20 ms after idle, while the clocks still
  // ramp, whichever kernel runs second looks faster.)
  if (cu_seqlens_k != nullptr && tiles <= 11 * items256) return AttnKernel::kIndependent128;
  // One round of the 128-row kernel against two: 1100 x 14 x 4 45.0 / 53.4, 300 x 14 x 10 16.9 / 23.4.
  if (items128 <= 2 * (int64_t)n_cus) return AttnKernel::kIndependent128;
  // A second round at most half full: 4096 x 22 170 / 190, x 24 176 / 211, 4000 x 24 178 / 197, 8000 x 12 334 / 404, 3841 x 23 161 /
  // 178, 2000 x 24 x 2 98 / 114, 1280 x 15 x 5 67 / 75, 1281 x 21 x 3 65 / 76, 8192, 300 and 77 x 12 350 / 418, 2458 and 1054 x 13 x
  // 2 98 / 114, against 1000 keys 4000 x 24 53 / 63;  past it 4352 x 24 234 / 230, 4352 x 26 243 / 233, 3000 x 36 170 / 166, 1500 x 22 x
  // 3 90 / 89, 8704 x 15 against 1000 keys 69.2 / 66.8.
  // Not self-attention of 12 to 18 key tiles: 1024 x 18 x 4 60.2 / 56.0, x 24 66.5 / 62.6, 900 x 20 x 4 55.5 / 52.3, 1100 x 19 x 4
  // 68.2 / 65.9, 1152 x 18 x 4 66.4 / 62.9, 800 x 16 x 6 50.7 / 47.8 (why sequences of about a
  // thousand rows take the 128-row kernel so long there is not known, 1280 x 19 x 4 is 67.1 / 75.6).  And with fewer tiles, where
  // either can be ahead, at most three sevenths full: 300 x 16 x 10 18.7 / 22.9, 410 x 16 x 10 29.7 / 31.4, 256 x 15 x 20 23.5 / 25.7,
  // 700 x 12 x 8 39.7 / 42.5, 512 x 16 x 9 35.9 / 36.1, 512 x 13 x 14 40.7 / 38.6, 640 x 13 x 9 42.6 / 38.6;  past it 410 x 16 x 12
  // 34.9 / 32.0, 512 x 16 x 12 41.5 / 38.2.
  const int64_t second = items256 - n_cus, third = items256 - 2 * (int64_t)n_cus;  // 256-row items of a round and later ones
  if (second > 0 && (tiles <= 11 * items256 ? 7 * second <= 3 * (int64_t)n_cus
                                            : 2 * second <= n_cus && (cu_seqlens_k != nullptr || tiles > 18 * items256)))
    return AttnKernel::kIndependent128;
  // A third round of equal items at most half full: 6000 x 24 387 / 413, 4096 x 33 264 / 278, x 40 298 / 317, 16384 x 10 1152 / 1202,
  // 2000 x 20 x 4 154 / 159, 1024 x 16 x 9 88 / 92, 700 x 24 x 8 63.4 / 65.9, 1000 x 16 x 10 90.5 / 90.9;  past it 2000 x 28 x 3 174 /
  // 171, 700 x 24 x 10 81 / 77, 6000 x 32 515 / 491, 16384 x 12 1389 / 1332.
  if (third > 0 && 2 * third <= n_cus && tiles == max_tiles * items256) return AttnKernel::kIndependent128;
  return AttnKernel::kPingPong256;
}

template <class P>
static hipError_t launch_p(const P& p, AttnKernel kernel, int head_dim, int n_cus, int32_t max_keys, hipStream_t stream) {
  const int64_t max_grid = (int64_t)n_cus * attn_fwd_wgs_per_cu(kernel, head_dim);
  const int grid = (int)(p.n_items < max_grid ? p.n_items : max_grid);
  if (kernel != AttnKernel::kIndependent128) {
    if (head_dim == 128) return launch_t<TilePP128, P, attn_fwd_pp_kernel<TilePP128, P>>(p, grid, stream);
    if (head_dim == 64) return launch_t<TilePP64, P, attn_fwd_pp_kernel<TilePP64, P>>(p, grid, stream);
  } else {
    // Where no compute unit has two items, D 128, us with two slots and a step's loads spread / at its start / with four slots:
    //   at most half of the compute units busy  448 x 8 9.5 / 10.1 / 10.5,  832 x 8 13.7 / 15.1 / 14.4,  1024 x 8 17.3 / 18.1 /
    //     17.1,  1280 x 10 20.6 / 21.5 / 20.1,  1536 x 10 23.6 / 24.8 / 22.9,  2048 x 8 29.4 / 31.4 / 28.4,  2048 x 3 27.1 / 30.3 /
    //     27.2,  4096 x 4 51.1 / 57.5 / 50.6: four from 16 tiles on, up to 4 % ahead;
    //   more of them  448 x 40 11.0 / 11.3 / 12.3,  700 x 24 14.7 / 15.0 / 15.7,  900 x 24 19.3 / 18.9 / 20.6,  1024 x 20 19.7 / 19.3 /
    //     19.5,  1024 x 24 21.2 / 20.8 / 21.6,  1152 x 24 23.2 / 23.4 / 24.2,  1280 x 24 25.7 / 26.4 / 26.0,  1792 x 17 32.0 / 33.7 /
    //     32.0,  3584 x 8 53.2 / 56.6 / 53.2: the loads at the start between 12 and 19 tiles, 2 % ahead (why is not known).
    if (head_dim == 128 && p.n_items <= (uint32_t)n_cus) {
      const bool half = 2 * p.n_items <= (uint32_t)n_cus;
      if (half && max_keys > 64 * 15) return launch_t<Tile128Deep, P, attn_fwd_kernel<Tile128Deep, P>>(p, grid, stream);
      if (!half && max_keys > 64 * 11 && max_keys <= 64 * 19)
        return launch_t<Tile128Burst, P, attn_fwd_kernel<Tile128Burst, P>>(p, grid, stream);
    }
    if (head_dim == 128) return launch_t<Tile128, P, attn_fwd_kernel<Tile128, P>>(p, grid, stream);
    if (head_dim == 64) return launch_t<Tile64, P, attn_fwd_kernel<Tile64, P>>(p, grid, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t attn_fwd_launch(const AttnParams& p, const PackList* list, AttnKernel kernel, int head_dim, int n_cus, int32_t max_keys,
                           hipStream_t stream) {
  if (list == nullptr) return launch_p(p, kernel, head_dim, n_cus, max_keys, stream);
  AttnListParams lp;
  static_cast<AttnParams&>(lp) = p;
  lp.list = *list;
  return launch_p(lp, kernel, head_dim, n_cus, max_keys, stream);
}

}  // namespace dit
