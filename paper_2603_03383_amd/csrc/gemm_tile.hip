// GEMM for more than 64 rows (several sequences verified together): sum_k X[m][k] * W[n][k], bf16 or fp16 in (element
// type E), fp32 out.  From ~100 rows on a weight is used often enough that the matrix cores, and the bytes a CU can
// request, matter as much as the HBM stream, so this kernel is built around operand reuse and a deep, barrier-light
// pipeline:
//   * a workgroup owns BM = 32 WR MT rows x BN = 32 WC NT columns (up to 256 x 128, so every weight is fetched once per
//     row block) and consists of TWO groups of WR x WC = 3, 4 or 6 waves; a round brings 64 features of X and W to LDS and
//     group g multiplies features 32g .. 32g + 31 of it.  The two groups share a CU's SIMDs, so one group's LDS reads
//     and waits overlap the other's MFMAs, and the K split inside the workgroup costs one exchange through LDS at the
//     end instead of a partial-sum slot in memory;
//   * both operands go straight to LDS (`global_load_lds`, 16 B per lane, no registers) into a ring of NS rounds; a wave
//     waits for its own loads of a round with a counted vmcnt and one workgroup barrier per round makes them everyone's.
//     The loads are written as inline assembly because the compiler, once it sees loads that write LDS, drains all
//     of them before every LDS read;
//   * the operands of a k-step are read from LDS while the previous k-step multiplies (two register sets), so that after a
//     barrier the matrix cores have work while all eight waves read LDS at once;
//   * X is read row-major, 128 B (one cache line) of eight rows per instruction; the 16-byte chunks of a row are XOR-ed
//     with the row number on the way in (through the per-lane source addresses), which spreads the operand reads over the
//     banks without padding (2.6 conflict cycles are counted per 16-byte read).  W arrives in the packed order (common.h): 4 KiB per tile and round, contiguous;
//   * the MFMA is issued as W x X^T: a lane then holds four consecutive output columns of ONE row per register quad, so
//     sums leave as 16-byte (fp32) or 8-byte (SwiGLU output) stores.
// What bounds it: below ~300 rows the loads (a CU takes in 45 - 62 GB/s of X and W whatever the ring holds, the chip some 10 TB/s: see
// BURSTS below), hence the tall tiles; at 1024 rows the LDS, which a round of the 256 x 128 tile asks for 96 KiB of
// operand reads and 48 KiB of incoming loads beside 1024 clocks of MFMAs (1024 x 22016 x 4096: 196 us; without the loads
// 145, without the MFMAs 146).  Measured on [M, K] x [N, K]^T, us per launch, before (128 x 256 tiles, operands through registers) / now:
// 192 rows: 12288 x 4096: 55 / 32, 22016 x 4096 (with SwiGLU): 88 / 50, 4096 x 4096: 20.6 / 16.4, 4096 x 11008: 38 / 30
// (35 / 58.7 / 17.2 / 32.1 without the second register set, 33.1 / 55.1 / 17.2 / 31.7 with the addresses of every load worked out
// anew; 1024 rows, likewise: 128 / 121 / 117, 206 / 196 / 187, 42 / 40.5 / 39, 108 / 101 / 97).
// 96 rows had no kernel but the portable one (800 / 24, 840 / 38, 810 / 12, 2170 / 23).
#include "gemm_rows.h"

namespace mdz {

typedef f32x16_t f32x16;
typedef u32x4_t u32x4;

// SWIGLU (gate/up matrix): an unsplit launch writes SiLU(gate) * up as E instead of the sums.  NT == 2: a wave's two tiles are the gate and
// the up columns of the same 32 features; NT == 1: its tile is 16 gate and the 16 up columns of 16 features, gathered by the load's lanes.
// DIRECT = false: X or W does not start on 16 bytes (a caller's buffer; the C interface asks for no alignment).  The same ring is
// filled through registers, from ordinary loads that are requested a round before they are written to LDS.  (128000 x 4096, us,
// aligned / not: 135 rows 217 / 329, 192 rows 228 / 344, 1024 rows 882 (gemm_wide.hip) / 1561; the portable kernel takes 3854, 3990, 18800.)
template <typename E, int WR, int WC, int MT, int NT, int NS, bool SWIGLU, bool DIRECT, bool BURSTS>
__global__ void __launch_bounds__(2 * WR * WC * 64, (2 * WR * WC + 3) / 4)
    gemm_tile_kernel(const E* __restrict__ X, int M, int K, const E* __restrict__ Wp, int n_tiles, float* __restrict__ P,
                     int64_t ldp, int64_t part_stride, int nb_m, int nb_n, int ksplit, E* __restrict__ U) {
  static_assert(!SWIGLU || NT <= 2, "a wave holds the gate and the up columns of its features: two tiles, or the halves of one");
  constexpr int GW = WR * WC, NW = 2 * GW;             // waves of a group and of the workgroup
  // X comes from L2 and W from HBM, but a CU's vector memory path returns in order and takes in no more from ~32 KiB of requests on, so X requests queued
  // among W requests take as long as those.  With a ring of four rounds the X of two rounds is requested in one round and the W of two
  // in the next: 24 + 16 KiB a round (192 x 128) then stream at 62 GB/s per CU instead of 56, 16 + 16 KiB at 52 instead of 48.
  // us per launch, mixed / in bursts: 192 rows, 22016 x 4096 52.3 / 50.9, 12288 x 4096 33.9 / 33.2; 128 rows, a step of 4 layers 814 / 793.
  // That holds where a round asks for about as much of X as of W and W comes from HBM.  Rows beyond M repeat a row and come at once, tiles of 64
  // columns ask for little W, and several row blocks share it through L2: there whole rounds are requested, up to four ahead (70 rows on
  // 128 x 128: 27648 x 5120 51.7 / 52.5, 15360 x 5120 32.3 / 32.9; 384 rows on 192 x 128, 4096 x 4096 and 4096 x 11008 32.8 / 33.3).
  static_assert(!BURSTS || (DIRECT && NS == 4), "bursts: the wait counts below are for a ring of four rounds");
  constexpr bool MIXED = SWIGLU && NT == 1;            // a tile is 16 gate and the 16 up columns of the same features
  constexpr int XT = WR * MT, WT = WC * NT;            // 32-row and 32-column tiles of the workgroup
  constexpr int UX = XT * 4, UT = (XT + WT) * 4;       // 1 KiB pieces of a round: X (8 rows x 128 B each), then W
  constexpr int LX = UX / NW, LW = WT * 4 / NW, L = LX + LW; // loads per wave and round
  static_assert(LX * NW == UX && L * NW == UT, "the waves share the pieces of a round evenly");
  constexpr uint32_t kSlot = UT * 1024;
  static_assert(NS * kSlot >= GW * MT * NT * 4096, "the groups' exchange fits the ring");
  extern __shared__ __attribute__((aligned(1024))) uint8_t lds_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Workgroups are dealt round-robin to the 8 XCDs: column blocks are dealt the same way and the row blocks of a column
  // block follow each other on one XCD, so they share its weights through that XCD's L2.
  const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
  const int bn = (seq / nb_m) * 8 + xcd, bm = seq % nb_m;
  if (bn >= nb_n) return;
  const int n_rounds = K / kRound;
  const int r_lo = (int)((int64_t)blockIdx.z * n_rounds / ksplit), r_hi = (int)((int64_t)(blockIdx.z + 1) * n_rounds / ksplit);
  const int nst256 = (K + kStageFeatures - 1) / kStageFeatures;
  const int grp = wave / GW, wg = wave % GW, wr = wg / WC, wc = wg % WC;

  f32x16 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const uint32_t lds0 = MDZ_LDS_ADDR(lds_raw);
  // Load cursor.  A load is two instructions and a wait state: addresses are a scalar base of X and of W, advanced by additions from round to
  // round, and per-lane offsets (from the block's first row) that do not change.  Rows beyond M re-read row M-1 and tiles beyond
  // n_tiles the block's first tile; neither is stored.  Past the range the cursor stays on its last round, which is not multiplied again, so the
  // wait counts below are the same in every trip.
  const int n = r_hi - r_lo;
  const int row0 = bm * XT * 32;
  uint32_t xoff[LX], woff[LW];
#pragma unroll
  for (int q = 0; q < LX; ++q) {
    const int row = min((q * NW + wave) * 8 + (lane >> 3), M - 1 - row0);
    xoff[q] = (uint32_t)row * (uint32_t)K * 2 + ((lane & 7) ^ (lane >> 3)) * 16;
  }
  // packed order [band of 4 tiles][stage of 256 features][tile in band][16 k-steps][lane]
  const int t0 = bn * WT, band0 = t0 >> 2;  // the block's first tile, and its band
#pragma unroll
  for (int q = 0; q < LW; ++q) {
    const int p = q * NW + wave, t = t0 + (p >> 2) < n_tiles ? t0 + (p >> 2) : t0;  // this wave loads k-step p % 4 of tile t in every round
    const int src = MIXED ? t & ~1 : t;  // (the up tile lies 16 KiB behind its gate tile)
    const uint32_t in_unit = MIXED ? ((t & 1) * 16 + (lane & 15) + (lane & 32)) * 16 + ((lane >> 4) & 1) * 16384 : lane * 16;
    woff[q] = (uint32_t)((src >> 2) - band0) * (uint32_t)nst256 * 65536u + (src & 3) * 16384 + (p & 3) * 1024 + in_unit;
  }
  const uint8_t* xp = reinterpret_cast<const uint8_t*>(X) + ((int64_t)row0 * K + (int64_t)r_lo * kRound) * 2;
  const uint8_t* wp = reinterpret_cast<const uint8_t*>(Wp) + ((int64_t)band0 * nst256 + (r_lo >> 2)) * 65536 + (r_lo & 3) * 4096;
  int next_x = r_lo, next_w = r_lo;
  typedef u32x4 u32x4_any __attribute__((aligned(2)));
  u32x4 held[DIRECT ? 1 : L];  // (through registers: the round after the newest one in LDS)
  auto load_x = [&](int slot) {  // requests the round under the X cursor, then advances it
    static_for<LX>([&](auto q) { load_to_lds<decltype(q)::value * NW * 1024>(xp, xoff[decltype(q)::value], lds0 + slot * kSlot + wave * 1024); });
    if (next_x + 1 < r_hi) ++next_x, xp += kRound * 2;
  };
  auto load_w = [&](int slot) {
    static_for<LW>([&](auto q) {
      load_to_lds<UX * 1024 + decltype(q)::value * NW * 1024, true>(wp, woff[decltype(q)::value], lds0 + slot * kSlot + wave * 1024);
    });
    if (next_w + 1 < r_hi) ++next_w, wp += (next_w & 3) ? 4096 : 4096 + 3 * 16384;
  };
  auto load_round = [&](int slot) {
    if constexpr (DIRECT) {
      load_x(slot);
      load_w(slot);
    } else {
      uint8_t* dst = lds_raw + slot * kSlot + wave * 1024 + lane * 16;
#pragma unroll
      for (int q = 0; q < L; ++q) *reinterpret_cast<u32x4*>(dst + (q < LX ? q * NW * 1024 : UX * 1024 + (q - LX) * NW * 1024)) = held[q];
    }
  };
  auto fetch_round = [&]() {  // (through registers)
    if constexpr (!DIRECT) {
#pragma unroll
      for (int q = 0; q < LX; ++q) held[q] = *reinterpret_cast<const u32x4_any*>(xp + xoff[q]);
#pragma unroll
      for (int q = 0; q < LW; ++q) held[LX + q] = *reinterpret_cast<const u32x4_any*>(wp + woff[q]);
      if (next_x + 1 < r_hi) {
        ++next_x;
        xp += kRound * 2, wp += (next_x & 3) ? 4096 : 4096 + 3 * 16384;
      }
    }
  };

  // Operands of one k-step (16 of the group's 32 features of a round), LDS -> registers, and their products.
  auto read_ops = [&](int slot, int ks, u32x4 (&a)[MT], u32x4 (&b)[NT]) {
    const uint8_t* base = lds_raw + slot * kSlot;
#pragma unroll
    for (int j = 0; j < NT; ++j)
      b[j] = *reinterpret_cast<const u32x4*>(base + (UX + (wc * NT + j) * 4 + grp * 2 + ks) * 1024 + lane * 16);
#pragma unroll
    for (int i = 0; i < MT; ++i)
      a[i] = *reinterpret_cast<const u32x4*>(base + ((wr * MT + i) * 32 + (lane & 31)) * 128 +
                                             ((grp * 4 + ks * 2 + (lane >> 5)) ^ (lane & 7)) * 16);
  };
  auto multiply = [&](const u32x4 (&a)[MT], const u32x4 (&b)[NT]) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[i][j] = Elem16<E>::mfma(b[j], a[i], acc[i][j]);
  };

  if constexpr (BURSTS) {
    load_x(0), load_x(1), load_w(0), load_w(1), load_w(2);
    wait_loads<2 * LW>();
  } else {
#pragma unroll
    for (int s = 0; s < NS - 1; ++s) {
      fetch_round();
      load_round(s);
    }
    if constexpr (DIRECT) {
      wait_loads<(NS - 2) * L>();
    } else {
      fetch_round();
      wait_lds();
    }
  }
  __builtin_amdgcn_s_barrier();  // round 0 is in LDS for everyone
  __builtin_amdgcn_sched_barrier(0);
  u32x4 a0[MT], b0[NT], a1[MT], b1[NT];
  read_ops(0, 0, a0, b0);
  int slot = 0;
  auto round = [&](auto odd) {  // multiplies the round in `slot`
    const int prev = slot == 0 ? NS - 1 : slot - 1, next = slot + 1 == NS ? 0 : slot + 1;
    read_ops(slot, 1, a1, b1);
    __builtin_amdgcn_sched_barrier(0);
    // (everyone had read the previous round before the last barrier)
    if constexpr (BURSTS) {
      if constexpr (decltype(odd)::value) load_w((slot + 2) & 3), load_w(prev);
      else load_x((slot + 2) & 3), load_x(prev);
    } else {
      load_round(prev);
      fetch_round();
    }
    __builtin_amdgcn_sched_barrier(0);
    multiply(a0, b0);
    __builtin_amdgcn_sched_barrier(0);
    wait_lds();  // this wave's reads of the slot are in registers before the barrier lets it be overwritten
    if constexpr (BURSTS) wait_loads<decltype(odd)::value ? LX + 2 * LW : LW + 2 * LX>();
    else if constexpr (DIRECT) wait_loads<(NS - 2) * L>();
    __builtin_amdgcn_s_barrier();  // the next round is in LDS for everyone, and everyone has read this one
    __builtin_amdgcn_sched_barrier(0);
    read_ops(next, 0, a0, b0);  // (behind the last round: a repeated one, never multiplied)
    __builtin_amdgcn_sched_barrier(0);
    multiply(a1, b1);
    __builtin_amdgcn_sched_barrier(0);
    slot = next;
  };
  for (int s = 0; s < n; s += 2) {
    round(std::false_type{});
    if (s + 1 < n) round(std::true_type{});
  }
  wait_lds();
  wait_loads<0>();
  __syncthreads();

  // The groups exchange halves through LDS: group 0 finishes the even row tiles, group 1 the odd ones (sums of group 0
  // first, whoever adds them).
  float* xch = reinterpret_cast<float*>(lds_raw);
  auto cell = [&](int i, int j, int q) { return xch + ((((i * NT + j) * 4 + q) * GW + wg) * 64 + lane) * 4; };
#pragma unroll
  for (int i = 0; i < MT; ++i)
    if ((i & 1) != grp) {
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(cell(i, j, q)) =
              float4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
    }
  __syncthreads();
  // D layout of W x X^T: lane holds row m = lane % 32 of the tile; register 4q + e is column 8q + 4 (lane / 32) + e.
  float* out = SWIGLU ? nullptr : P + (int64_t)blockIdx.z * part_stride;
#pragma unroll
  for (int i = 0; i < MT; ++i)
    if ((i & 1) == grp) {
      const int m = (bm * XT + wr * MT + i) * 32 + (lane & 31);
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 o = *reinterpret_cast<const float4*>(cell(i, j, q));
          acc[i][j][4 * q] += o.x, acc[i][j][4 * q + 1] += o.y, acc[i][j][4 * q + 2] += o.z, acc[i][j][4 * q + 3] += o.w;
        }
      if (m >= M) continue;
      if constexpr (SWIGLU) {
        // NT == 2: gate tile `tile`, its features are 16 tile .. + 31 of [M][16 n_tiles]; MIXED: features 16 tile .. + 15
        const int tile = t0 + wc * NT;
        if (tile + NT - 1 < n_tiles) {
          E* u = U + (int64_t)m * (n_tiles * 16) + tile * 16 + 4 * (lane >> 5);
#pragma unroll
          for (int q = 0; q < 2 * NT; ++q) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = silu_tile(acc[i][0][4 * q + e]) * (MIXED ? acc[i][0][4 * (q + 2) + e] : acc[i][NT - 1][4 * q + e]);
            *reinterpret_cast<uint2*>(u + 8 * q) = uint2{Elem16<E>::pack2(v[0], v[1]), Elem16<E>::pack2(v[2], v[3])};
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          const int tile = t0 + wc * NT + j;
          if (tile < n_tiles) {
            float* o = out + (int64_t)m * ldp + tile * 32 + 4 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 4; ++q)
              *reinterpret_cast<float4*>(o + 8 * q) =
                  float4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          }
        }
      }
    }
}

namespace {
struct TilePlan {
  int bm, bn, ksplit;  // rows and columns of a workgroup's tile, K splits
  int nb_m, nb_n;
  double us;  // modelled
};

// Tile and split by a small model of the launch: a workgroup's time is the larger of its requests at 50 GB/s and its
// MFMAs at 4.5 TFLOP/s (what a CU sustains in this kernel's loop on real data) plus ~4 us of start and tail, workgroups run
// in rounds of one per CU, the launch cannot beat the HBM stream of W, and every partial-sum slot is written here and read
// back by the consumer.  The constants are measured on MI355X; the choice only moves work between equal results.
// The tiles of 96 columns are for a single row block, and only where they put a workgroup on at least 7/8 of the CUs, no CU having two:
// us per launch, 128 / 96 columns: 90 rows x 22016 x 4096 (172 / 230 workgroups) 40.6 / 38.4, x 12288 x 4096 (192 / 256) 26.7 / 24.7, 192 rows
// 51.9 / 50.6 and 33.8 / 32.1; elsewhere they lose: 90 rows x 4096 x 11008 (224 / 215) 23.3 / 25.6, 80 rows of a 5120-wide layer +5.
TilePlan plan_tile(int M, int N, int K, int max_split, bool swiglu) {
  TilePlan best{};
  double best_t = 1e30;
  const int n_rounds = K / kRound, cus = num_cus();
  const int shapes[][2] = {{96, 96}, {128, 128}, {128, 64}, {192, 128}, {192, 96}, {192, 64}, {256, 128}, {256, 64}};
  for (auto& sh : shapes) {
    const int bm = sh[0], bn = sh[1];
    if ((swiglu && bn < 96) || (bn == 96 && M > bm)) continue;
    const int nb_m = (M + bm - 1) / bm, nb_n = (N + bn - 1) / bn;
    for (int ks = 1; ks <= 8 && ks <= max_split && ks <= n_rounds; ++ks) {
      const int64_t wgs = (int64_t)nb_m * nb_n * ks;
      if (bn == 96 && (wgs > cus || wgs * 8 < cus * 7)) continue;
      const double feats = (double)((n_rounds + ks - 1) / ks) * kRound;
      const double load = feats * (bm + bn) * 2 / 50e3, mfma = feats * bm * bn * 2 / 4.5e6;  // us
      const double rounds = (double)((wgs + cus - 1) / cus);
      double t = rounds * ((load > mfma ? load : mfma) + 4.0);
      const double hbm = (double)N * K * 2 / 5.5e6 + 4.0;
      if (t < hbm) t = hbm;
      t += (double)ks * M * N * 4 * (1.0 / 5e6 + 1.0 / 4e6);
      if (t < best_t - 1e-9) best_t = t, best = TilePlan{bm, bn, ks, nb_m, nb_n, t};
    }
  }
  return best;
}
}  // namespace

bool gemm_tile_supported(int dtype, int M, int N, int K) {
  // (K: the byte offset of a row of a 256-row block is kept in 32 bits)
  return is_16bit(dtype) && M > 64 && N % 32 == 0 && K % kRound == 0 && K >= kRound && K <= 1 << 22;
}

double gemm_tile_cost(int M, int N, int K, int max_split, bool swiglu, int* slots) {
  const TilePlan p = plan_tile(M, N, K, max_split, swiglu);
  if (slots) *slots = p.ksplit;
  return p.us;
}

ManyRowsPlan gemm_tile_plan(int M, int N, int K, int max_split, bool swiglu) {
  const TilePlan p = plan_tile(M, N, K, max_split, swiglu);
  return ManyRowsPlan{false, p.bm, p.bn, p.ksplit};
}

// partial-sum slots launch_gemm_tile will write for this problem (sizes the slot workspace)
int gemm_tile_slots(int M, int N, int K, int max_split) {
  int slots = 1;
  if (gemm_wide_preferred(M, N, K, max_split, false)) gemm_wide_cost(M, N, K, max_split, false, &slots);
  else gemm_tile_cost(M, N, K, max_split, false, &slots);
  return slots;
}

template <typename E, bool SWIGLU, bool DIRECT>
static int launch_gemm_tile_t(const void* X, const void* Wp, float* P, int M, int N, int K, int64_t ldp, int64_t part_stride,
                              int max_split, Partials* res, void* U, hipStream_t st) {
  const TilePlan p = plan_tile(M, N, K, max_split, SWIGLU);
  if (res) {
    res->n = p.ksplit;
    res->split_grid = 0;
    res->band_cols = p.bn;
    res->n_stages = 1;
    res->split_units = 0;
  }
  const dim3 grid((p.nb_n + 7) / 8 * 8 * p.nb_m, 1, p.ksplit);
  // X and W in bursts (see the kernel): one row block, at least four fifths as many rows as columns
  const bool full = p.nb_m == 1 && 5 * M >= 4 * p.bn;
#define MDZ_TILE_CASE(WR, WC, MT, NT, NS, BURSTS, TAKEN)                                                                  \
  if (p.bm == 32 * WR * MT && p.bn == 32 * WC * NT && (TAKEN)) {                                                          \
    constexpr int lds_bytes = NS * (WR * MT + WC * NT) * 4 * 1024;                                                        \
    static_assert(lds_bytes <= 160 * 1024, "LDS of a CU");                                                                \
    constexpr auto kernel = gemm_tile_kernel<E, WR, WC, MT, NT, NS, SWIGLU, DIRECT, DIRECT && BURSTS>;                    \
    MDZ_SET_LDS_ONCE(kernel, lds_bytes);                                                                                  \
    launch_timed(PROF_GEMM_LARGE, kernel, grid, 2 * WR * WC * 64, lds_bytes, st, (const E*)X, M, K, (const E*)Wp, N / 32, P, ldp, \
                 part_stride, p.nb_m, p.nb_n, p.ksplit, (E*)U);                                                           \
    MDZ_LAUNCH_CHECK();                                                                                                   \
    return MDZ_OK;                                                                                                        \
  }
  MDZ_TILE_CASE(1, 3, 3, 1, 4, true, true)
  MDZ_TILE_CASE(2, 3, 3, 1, 4, true, true)
  if constexpr (DIRECT) MDZ_TILE_CASE(2, 2, 2, 2, 4, true, full)
  MDZ_TILE_CASE(2, 2, 2, 2, 4, false, true)
  if constexpr (DIRECT) MDZ_TILE_CASE(2, 2, 3, 2, 4, true, full)
  MDZ_TILE_CASE(2, 2, 3, 2, 3, false, true)
  MDZ_TILE_CASE(2, 2, 4, 2, 3, false, true)
  if constexpr (!SWIGLU) {
    MDZ_TILE_CASE(2, 2, 2, 1, 5, false, true)
    MDZ_TILE_CASE(2, 2, 3, 1, 4, false, true)
    MDZ_TILE_CASE(2, 2, 4, 1, 4, false, true)
  }
#undef MDZ_TILE_CASE
  MDZ_FAIL(MDZ_EUNSUPPORTED, "gemm: no tile kernel for a %d x %d tile", p.bm, p.bn);
}

static bool starts_on_16(const void* X, const void* Wp) {  // what the direct-to-LDS loads need
  return ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Wp)) & 15) == 0;
}

int launch_gemm_tile(int dtype, const void* X, const void* Wp, float* P, int M, int N, int K, int64_t ldp,
                     int64_t part_stride, int max_split, Partials* res, hipStream_t st) {
  if (!starts_on_16(X, Wp)) {
    max_split = gemm_tile_slots(M, N, K, max_split);  // (the buffer is sized for the plan of aligned operands)
    MDZ_WITH_ELEM16(dtype, return (launch_gemm_tile_t<E, false, false>(X, Wp, P, M, N, K, ldp, part_stride, max_split, res, nullptr, st)));
  }
  if (gemm_wide_preferred(M, N, K, max_split, false))
    return launch_gemm_wide(dtype, X, Wp, P, M, N, K, ldp, part_stride, max_split, res, st);
  MDZ_WITH_ELEM16(dtype, return (launch_gemm_tile_t<E, false, true>(X, Wp, P, M, N, K, ldp, part_stride, max_split, res, nullptr, st)));
}

// gate/up GEMM with the SwiGLU in its epilogue: U [M][N / 2] of the storage type
bool gemm_tile_swiglu_supported(int dtype, int M, int N, int K) { return gemm_tile_supported(dtype, M, N, K) && N % 64 == 0; }

int launch_gemm_tile_swiglu(int dtype, const void* X, const void* Wp, void* U, int M, int N, int K, hipStream_t st) {
  if (!starts_on_16(X, Wp))
    MDZ_WITH_ELEM16(dtype, return (launch_gemm_tile_t<E, true, false>(X, Wp, nullptr, M, N, K, N, 0, 1, nullptr, U, st)));
  if (gemm_wide_preferred(M, N, K, 1, true)) return launch_gemm_wide_swiglu(dtype, X, Wp, U, M, N, K, st);
  MDZ_WITH_ELEM16(dtype, return (launch_gemm_tile_t<E, true, true>(X, Wp, nullptr, M, N, K, N, 0, 1, nullptr, U, st)));
}

}  // namespace mdz
