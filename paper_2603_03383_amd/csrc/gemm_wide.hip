// GEMM for many rows (several sequences on the 64-node tree), where the matrix cores are the bound: sum_k X[m][k] * W[n][k],
// bf16 or fp16 in (element type E), fp32 out.  Rows tiles of 192 or 256 x 256 columns, four waves of up to 128 x 128 each (all
// 256 accumulation registers of a lane), one wave per SIMD: the largest tile a CU can hold asks for the fewest LDS and L2 bytes
// per product (a round of 64 features: 128 KiB of operand reads and 64 KiB of loads beside 2048 clocks of MFMAs; the 256 x 128
// tile of gemm_tile.hip needs 288 KiB for the same work and is bound by that).
//   * Loads go straight to LDS: X in a ring of three rounds (row-major, a cache line of eight rows per load, 16-byte chunks
//     XOR-ed with the row number), W in a ring of four half rounds (packed order, common.h), 160 KiB together.
//   * With one wave per SIMD nothing hides an instruction but the MFMA in front of it (32 clocks), so the loop is laid out by
//     hand: behind every MFMA at most one LDS read and one load, a load being two instructions and a wait state; operands are read one
//     k-step ahead.  (Address arithmetic per load and loads in bunches cost 3970 clocks per round instead of 2660.)
//   * A workgroup runs several bands of 256 columns one after the other without emptying the rings, or a K split of one band.
// What bounds it now: power.  The clock falls from 2.4 to ~1.65 GHz and the loop then runs at 75 % of the MFMA rate of that
// clock; fewer busy CUs run faster, so a launch takes no more of them than its rounds need.  Measured, us per launch, gemm_tile / this one:
// 1024 rows: 12288 x 4096: 117 / 100 (and one partial sum instead of two), 22016 x 4096 with SwiGLU: 187 / 178, 128000 x 4096:
// 1082 / 957 (1.12 PFLOP/s); 512 rows: 65 / 58, 118 / 101, 602 / 539; 320 rows: 48 / 46, 95 / 84, 476 / 435.  (The choice between the
// two is by modelled times, which are close at some of these: at 512 rows they put 12288 x 4096 on gemm_tile, 78.2 us against 79.1.)
#include "gemm_rows.h"

namespace mdz {

typedef f32x16_t f32x16;
typedef u32x4_t u32x4;

namespace {
__device__ inline void workgroup_barrier() {
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}
}  // namespace

// SWIGLU (gate/up matrix, whole bands): of a wave's four tiles 0, 2 are gate and 1, 3 the up columns of the same features;
// SiLU(gate) * up is written as E instead of the sums.
// ARGMAX (LM head of a verify pass that wants no logits, whole bands): a lane keeps the best (value, column) of its rows over the
// workgroup's bands; two candidates per row and workgroup leave the kernel instead of the sums.
template <typename E, int MT, bool SWIGLU, bool ARGMAX>
__global__ void __launch_bounds__(256, 1)
    gemm_wide_kernel(const E* __restrict__ X, int M, int K, const E* __restrict__ Wp, int n_tiles, float* __restrict__ P,
                     int64_t ldp, int64_t part_stride, int nb_m, int nb_n, int G, int ksplit, E* __restrict__ U, ArgCand* __restrict__ cand) {
  constexpr int NT = 4, BM = 64 * MT;
  constexpr int LX = 2 * MT, LW = 4;                // loads of a wave: X of one round, W of half a round
  constexpr int HX = MT, LWIN = LW + HX;            // a window: W of half a round and half of a round's X
  constexpr int SP = MT * NT * 2 / LWIN;            // MFMAs from one load to the next
  constexpr int LSEG = MT * NT / SP;                // loads in the first half of a window, the rest follows in the second
  static_assert(LSEG <= LWIN && LWIN <= 2 * LSEG, "every load of a window has its place");
  constexpr uint32_t kXSlot = BM * 128, kWSlot = 16 * 1024;
  constexpr uint32_t kW0 = 3 * kXSlot;              // X ring of three rounds, then W ring of four half rounds
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (block order: see gemm_tile.hip)
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int w = (seq / nb_m) * 8 + xcd, bm = seq % nb_m;
  if (w >= G) return;
  const int n_rounds = K / kRound;
  int u_lo, u_hi;  // units: band after band, n_rounds each
  if (ksplit > 1) {  // (G == nb_n * ksplit) one band, a part of its rounds
    const int band = w / ksplit, z = w % ksplit;
    u_lo = band * n_rounds + z * n_rounds / ksplit, u_hi = band * n_rounds + (z + 1) * n_rounds / ksplit;
  } else {  // whole bands
    u_lo = (int)((int64_t)w * nb_n / G) * n_rounds, u_hi = (int)((int64_t)(w + 1) * nb_n / G) * n_rounds;
  }
  if (u_lo >= u_hi) return;
  const int nst256 = (K + kStageFeatures - 1) / kStageFeatures;
  const int wr = wave >> 1, wc = wave & 1;

  f32x16 acc[MT][NT];
  auto zero_acc = [&]() {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  };
  zero_acc();
  const uint32_t lds0 = MDZ_LDS_ADDR(lds_raw);
  // Load cursors.  A load is two instructions (m0, load) and a wait state: addresses are a scalar base per round or half round, advanced by
  // additions, and per-lane offsets that do not change.  A cursor stays on the range's last piece when it gets there.
  const int64_t bs = (int64_t)nst256 * 65536;  // bytes of a band of 128 columns
  X += (int64_t)bm * BM * K;  // the block's first row: offsets are relative to it
  uint32_t xoff[LX], woff[LW];
#pragma unroll
  for (int q = 0; q < LX; ++q) {
    const int row = min((q * 4 + wave) * 8 + (lane >> 3), M - 1 - bm * BM);
    xoff[q] = (uint32_t)row * (uint32_t)K * 2 + ((lane & 7) ^ (lane >> 3)) * 16;
  }
  int xr = u_lo % n_rounds, x_left = u_hi - u_lo - 1;
  const E* xp = X + xr * kRound;
  uint32_t x_lds = lds0 + wave * 1024;
  int wb = u_lo / n_rounds, wh = 2 * xr, w_left = 2 * (u_hi - u_lo) - 1;
  const uint8_t* wp;
  uint32_t w_lds = lds0 + kW0 + wave * 1024;
  auto w_band = [&]() {  // base and offsets of band wb from half round wh on; a missing second half of the band repeats the first
    wp = reinterpret_cast<const uint8_t*>(Wp) + wb * 2 * bs + (int64_t)(wh >> 3) * 65536 + (wh & 7) * 2048 + (wave >> 1) * 16384 +
         (wave & 1) * 1024;
    const uint32_t second = wb * 8 + 4 < n_tiles ? (uint32_t)bs : 0;
#pragma unroll
    for (int q = 0; q < LW; ++q) woff[q] = lane * 16 + (q & 1) * 32768 + (q >> 1) * second;
  };
  w_band();
  auto load_x = [&](auto q) { load_to_lds<decltype(q)::value * 4096>(xp, xoff[decltype(q)::value], x_lds); };
  auto load_w = [&](auto q) { load_to_lds<decltype(q)::value * 4096>(wp, woff[decltype(q)::value], w_lds); };
  auto next_x = [&]() {
    if (x_left > 0) {
      --x_left, ++xr, xp += kRound;
      if (xr == n_rounds) xr = 0, xp = X;
    }
    x_lds = x_lds == lds0 + 2 * kXSlot + wave * 1024 ? lds0 + wave * 1024 : x_lds + kXSlot;
  };
  auto next_w = [&]() {
    if (w_left > 0) {
      --w_left, ++wh, wp += 2048;
      if ((wh & 7) == 0) wp += 65536 - 16384;
      if (wh == 2 * n_rounds) wh = 0, ++wb, w_band();
    }
    w_lds = w_lds == lds0 + kW0 + 3 * kWSlot + wave * 1024 ? lds0 + kW0 + wave * 1024 : w_lds + kWSlot;
  };
  auto read_a = [&](int xslot, int c0, int i) {
    return *reinterpret_cast<const u32x4*>(lds_raw + xslot * kXSlot + ((wr * MT + i) * 32 + (lane & 31)) * 128 +
                                           ((c0 + (lane >> 5)) ^ (lane & 7)) * 16);
  };
  auto read_b = [&](int wslot, int ks, int j) {
    return *reinterpret_cast<const u32x4*>(lds_raw + kW0 + wslot * kWSlot + ((wc * NT + j) * 2 + ks) * 1024 + lane * 16);
  };

  int cb = u_lo / n_rounds, cr = u_lo % n_rounds;
  float best_v[MT];
  int best_i[MT];
#pragma unroll
  for (int i = 0; i < MT; ++i) best_v[i] = -INFINITY, best_i[i] = kNoIndex;
  auto flush = [&]() {
    float* out = SWIGLU || ARGMAX ? nullptr : P + (int64_t)(w % ksplit) * part_stride;
    auto pin = [&]() {  // holds the sums in accumulation registers until each is wanted; read out all at once they spill
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) asm volatile("" : "+a"(acc[i][j]));
    };
    pin();
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = bm * BM + (wr * MT + i) * 32 + (lane & 31);
      if constexpr (ARGMAX) {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          pin();
          const int tile = cb * 8 + wc * NT + j;
          if (tile < n_tiles) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int col = tile * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
              if (precedes(acc[i][j][r], col, best_v[i], best_i[i])) best_v[i] = acc[i][j][r], best_i[i] = col;
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        continue;
      }
      if (m >= M) continue;
      if constexpr (SWIGLU) {
#pragma unroll
        for (int jp = 0; jp < NT; jp += 2) {
          const int tile = cb * 8 + wc * NT + jp;
          pin();
          if (tile + 1 < n_tiles) {
            E* u = U + (int64_t)m * (n_tiles * 16) + tile * 16 + 4 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              float v[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = silu_tile(acc[i][jp][4 * q + e]) * acc[i][jp + 1][4 * q + e];
              *reinterpret_cast<uint2*>(u + 8 * q) = uint2{Elem16<E>::pack2(v[0], v[1]), Elem16<E>::pack2(v[2], v[3])};
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const int tile = cb * 8 + wc * NT + j;
          if (tile < n_tiles) {
            float* o = out + (int64_t)m * ldp + tile * 32 + 4 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 4; ++q)
              *reinterpret_cast<float4*>(o + 8 * q) =
                  float4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    zero_acc();
  };

  // A window is the stretch of MFMAs from one barrier to the next; it requests one W half round and half an X round, one load
  // every few MFMAs (in bunches they hold up the wave's MFMAs).  Window h, behind the barrier inside half round h, loads W half
  // h + 4 and, for h = 2 m + 1, the first half of X round m + 3, for h = 2 m the second half of X round m + 2: what the barrier of
  // half h hands over was requested in window h - 3 or before, so two windows stay in flight.
  auto load_piece = [&](auto ic, auto sec) {  // i-th load of a window: W and X pieces alternate
    constexpr int i = decltype(ic)::value;
    constexpr bool second = decltype(sec)::value;
    if constexpr (i >= 2 * HX) load_w(std::integral_constant<int, i - HX>{});
    else if constexpr (i & 1) load_x(std::integral_constant<int, (i >> 1) + (second ? HX : 0)>{});
    else load_w(std::integral_constant<int, (i >> 1)>{});
  };
  constexpr std::false_type first_half{};
  constexpr std::true_type second_half{};
  constexpr std::integral_constant<int, 0> first_part{};
  constexpr std::integral_constant<int, LSEG> second_part{};
  // before the loop: W 0 and X 0, then the windows of W 1, W 2 and the first part of the one of W 3
  static_for<LW>(load_w);
  static_for<LX>(load_x);
  next_w();
  next_x();
  static_for<LWIN>([&](auto i) { load_piece(i, first_half); });
  next_w();
  static_for<LWIN>([&](auto i) { load_piece(i, second_half); });
  next_w();
  next_x();
  static_for<LSEG>([&](auto i) { load_piece(i, first_half); });
  wait_loads<2 * LWIN + LSEG>();
  workgroup_barrier();
  u32x4 a0[MT], b0[NT], a1[MT], b1[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) a0[i] = read_a(0, 0, i);
#pragma unroll
  for (int j = 0; j < NT; ++j) b0[j] = read_b(0, 0, j);

  // The products of one k-step (a, b); meanwhile the operands of the next are read (na, nb) and part of a window is requested.
  auto segment = [&](const u32x4 (&a)[MT], const u32x4 (&b)[NT], u32x4 (&na)[MT], u32x4 (&nb)[NT], int xs, int chunk, int ws, int ks,
                     auto part, auto half) {
    static_for<MT * NT>([&](auto tc) {
      constexpr int t = decltype(tc)::value, load = decltype(part)::value + t / SP;
      acc[t / NT][t % NT] = Elem16<E>::mfma(b[t % NT], a[t / NT], acc[t / NT][t % NT]);
      if constexpr (t < MT) na[t] = read_a(xs, chunk, t);
      else if constexpr (t < MT + NT) nb[t - MT] = read_b(ws, ks, t - MT);
      if constexpr (t % SP == SP / 2 && load < LWIN) load_piece(std::integral_constant<int, load>{}, half);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // This wave's reads are in registers and its share of the next half round is in LDS, then everyone's.
  auto hand_over = [&]() {
    wait_lds();
    wait_loads<2 * LWIN>();
    workgroup_barrier();
  };

  int xslot = 0, wslot = 0;
  int left = u_hi - u_lo;
  while (left > 0) {  // a band, or the part of it that is this workgroup's
    int seg = min(left, n_rounds - cr);
    left -= seg;
    do {
      const int xnext = xslot == 2 ? 0 : xslot + 1;
      // even half: k-steps 0 and 1 (the barrier: its W half and the slots read so far are free, the next half is in LDS)
      segment(a0, b0, a1, b1, xslot, 2, wslot, 1, second_part, first_half);
      next_w();
      hand_over();
      segment(a1, b1, a0, b0, xslot, 4, (wslot + 1) & 3, 0, first_part, second_half);
      // odd half: k-steps 2 and 3
      segment(a0, b0, a1, b1, xslot, 6, (wslot + 1) & 3, 1, second_part, second_half);
      next_w();
      next_x();
      hand_over();
      segment(a1, b1, a0, b0, xnext, 0, (wslot + 2) & 3, 0, first_part, first_half);
      xslot = xnext;
      wslot = (wslot + 2) & 3;
      asm volatile("" : "+s"(seg));  // (keeps the compiler from folding the two loops and the flush's registers into one)
    } while (--seg > 0);
    flush();
    cr = 0, ++cb;
  }
  if constexpr (ARGMAX) {
#pragma unroll
    for (int i = 0; i < MT; ++i) {
      const int m = bm * BM + (wr * MT + i) * 32 + (lane & 31);
      const float ov = __shfl_xor(best_v[i], 32, 64);  // the row's other columns
      const int oi = __shfl_xor(best_i[i], 32, 64);
      if (precedes(ov, oi, best_v[i], best_i[i])) best_v[i] = ov, best_i[i] = oi;
      if (lane < 32 && m < M) cand[(int64_t)m * (2 * G) + 2 * w + wc] = ArgCand{best_v[i], best_i[i]};
    }
  }
  wait_lds();
  wait_loads<0>();  // no load may write LDS after the workgroup has given it back
}

namespace {
struct WidePlan {
  int mt, nb_m, nb_n, G, ksplit;  // G workgroups per row block
  double us;                      // modelled
};

// Rows per tile and split by a small model, measured on MI355X: a round takes 1.42 us (256 rows) or 1.15 us (192) on a few CUs
// and 1.2 times that on all (the clock falls), a launch ~7 us of start and tail, a further band ~3 us of stores; the launch cannot beat
// the HBM stream of W, and every partial-sum slot is written here and read back by the consumer.  Within the rounds that the
// busiest workgroup runs, as few workgroups as possible.
WidePlan plan_wide(int M, int N, int K, int max_split, bool swiglu) {
  WidePlan best{};
  best.us = 1e30;
  const int n_rounds = K / kRound, cus = num_cus(), nb_n = (N + 255) / 256;
  for (int mt = 3; mt <= 4; ++mt) {
    const int nb_m = (M + 64 * mt - 1) / (64 * mt), g_max = cus > nb_m ? cus / nb_m : 1;
    for (int ks = 1; ks <= n_rounds && ks <= max_split && (ks == 1 || nb_n * ks <= g_max); ++ks) {
      const int bands = ks == 1 ? (nb_n + g_max - 1) / g_max : 1;
      const int G = ks == 1 ? (nb_n + bands - 1) / bands : nb_n * ks;
      const double wgs = (double)nb_m * G, gens = wgs > cus ? (double)(((int64_t)nb_m * G + cus - 1) / cus) : 1.0;
      const double busy = wgs < cus ? wgs / cus : 1.0, round = (mt == 4 ? 1.42 : 1.15) * (0.75 + 0.45 * busy);
      double t = gens * ((double)bands * ((n_rounds + ks - 1) / ks) * round + 7.0 + (swiglu ? 0.0 : 3.0 * (bands - 1)));
      const double hbm = (double)N * K * 2 / 5e6 + 4.0;
      if (t < hbm) t = hbm;
      t += (double)ks * M * N * 4 * (1.0 / 5e6 + 1.0 / 4e6);
      if (t < best.us - 1e-9) best = WidePlan{mt, nb_m, nb_n, G, ks, t};
    }
  }
  return best;
}
}  // namespace

double gemm_wide_cost(int M, int N, int K, int max_split, bool swiglu, int* slots) {
  const WidePlan p = plan_wide(M, N, K, max_split, swiglu);
  if (slots) *slots = p.ksplit;
  return p.us;
}

ManyRowsPlan gemm_wide_plan(int M, int N, int K, int max_split, bool swiglu) {
  const WidePlan p = plan_wide(M, N, K, max_split, swiglu);
  return ManyRowsPlan{true, 64 * p.mt, 256, p.ksplit};
}

template <typename E, bool SWIGLU, bool ARGMAX = false>
static int launch_gemm_wide_t(const void* X, const void* Wp, float* P, int M, int N, int K, int64_t ldp, int64_t part_stride,
                              int max_split, Partials* res, void* U, hipStream_t st, ArgCand* cand = nullptr) {
  const WidePlan p = plan_wide(M, N, K, max_split, SWIGLU);
  if (res) {
    res->n = p.ksplit;
    res->split_grid = 0;
    res->band_cols = 256;
    res->n_stages = 1;
    res->split_units = 0;
  }
  const dim3 grid((p.G + 7) / 8 * 8 * p.nb_m);
#define MDZ_WIDE_CASE(MT)                                                                                                  \
  if (p.mt == MT) {                                                                                                        \
    constexpr int lds_bytes = 3 * 64 * MT * 128 + 4 * 16 * 1024;                                                           \
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");                                                                 \
    MDZ_SET_LDS_ONCE((gemm_wide_kernel<E, MT, SWIGLU, ARGMAX>), lds_bytes);                                                        \
    launch_timed(PROF_GEMM_LARGE, gemm_wide_kernel<E, MT, SWIGLU, ARGMAX>, grid, 256, lds_bytes, st, (const E*)X, M, K, (const E*)Wp, \
                 N / 32, P, ldp, part_stride, p.nb_m, p.nb_n, p.G, p.ksplit, (E*)U, cand);                                 \
    MDZ_LAUNCH_CHECK();                                                                                                    \
    return MDZ_OK;                                                                                                         \
  }
  MDZ_WIDE_CASE(3)
  MDZ_WIDE_CASE(4)
#undef MDZ_WIDE_CASE
  MDZ_FAIL(MDZ_EUNSUPPORTED, "gemm: no wide kernel for %d rows per tile", 64 * p.mt);
}

int launch_gemm_wide(int dtype, const void* X, const void* Wp, float* P, int M, int N, int K, int64_t ldp, int64_t part_stride,
                     int max_split, Partials* res, hipStream_t st) {
  MDZ_WITH_ELEM16(dtype, return (launch_gemm_wide_t<E, false>(X, Wp, P, M, N, K, ldp, part_stride, max_split, res, nullptr, st)));
}

int launch_gemm_wide_swiglu(int dtype, const void* X, const void* Wp, void* U, int M, int N, int K, hipStream_t st) {
  MDZ_WITH_ELEM16(dtype, return (launch_gemm_wide_t<E, true>(X, Wp, nullptr, M, N, K, N, 0, 1, nullptr, U, st)));
}

// The LM head of a verify pass when only the per-row argmax is wanted: cand receives M x gemm_wide_argmax_cands(...) candidates.
bool gemm_wide_argmax_supported(int dtype, int M, int N, int K) {
  return gemm_tile_supported(dtype, M, N, K) && gemm_wide_preferred(M, N, K, 1, false);
}
int gemm_wide_argmax_cands(int M, int N, int K) { return 2 * plan_wide(M, N, K, 1, false).G; }

int launch_gemm_wide_argmax(int dtype, const void* X, const void* Wp, int M, int N, int K, ArgCand* cand, hipStream_t st) {
  MDZ_WITH_ELEM16(dtype, return (launch_gemm_wide_t<E, false, true>(X, Wp, nullptr, M, N, K, 0, 0, 1, nullptr, nullptr, st, cand)));
}

}  // namespace mdz
