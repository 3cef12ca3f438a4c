// Tree-masked attention for 16-bit storage (bf16 or fp16, element type E), trees of 64 or 15 nodes, head_dim 128, on gfx950 MFMA
// (Section 3.2: all T candidates attend in one pass; node i sees the whole prefix plus the tree slots
// its row of the static visibility matrix allows).
//
// One workgroup = 4 waves handles one (sequence, head, key-split).  All 64 queries ride along every
// key, so K and V are read from HBM exactly once per head.  A wave walks 32-key blocks of the tiled
// cache (common.h): each 1 KiB unit is loaded with one contiguous 16-byte-per-lane load and used
// directly as an MFMA A operand.  Scores are computed transposed (keys x queries), which leaves every
// lane with 16 keys of ONE query: the running max / sum need a single exchange with lane+32, and the
// probabilities are packed to the storage type in place as the B operand of the second MFMA (out^T = V^T P^T).
// The tree mask is one 64-bit word per query (a compile-time table) tested only in blocks that reach
// past the prefix.  Waves merge through LDS, key-splits through a small second kernel, both in a fixed
// order, so results are deterministic.
// Q8 = true: the cache holds 8-bit rows (E4M3 codes + one fp32 scale per row, common.h).  A block is then 4 K units,
// 4 V units and 2 x 32 scales; codes convert exactly to the 16-bit element type in registers (two k-steps per 16-byte
// load), the K scales multiply the scores and the V scales the probabilities, both in fp32, so the MFMAs are the same.
// Key-splits: when the kernel starts from the QKV partial sums, the last split owns every block that holds a
// tree slot (it is the one that has to produce those K / V rows first) and the other splits share the blocks
// that hold prefix keys only, which need nothing but Q: the longer prologue (three matrices reduced instead of one) then
// falls on a workgroup with few blocks instead of one with an even share of the prefix.
#include <type_traits>

#include "kernels.h"

namespace mdz {

typedef f32x16_t f32x16;
typedef u32x4_t u32x4;

constexpr int kHD = 128;         // head_dim
constexpr int kQRow = kHD * 2 + 16;  // bytes per staged Q row
constexpr float kLazyLog2 = 8.f;  // see the key loop: how far a block's maximum may exceed the running reference

// F features of one row of one head's q, k or v in the QKV GEMM output, and their rotary partners 64 columns on.  load() requests
// the first two partial-sum slots so that the loads of several of these can be in flight together; sum() adds the slots in order
// and fetches what lies beyond, one slot after the other.  (A product of 3 x 4096 or 3 x 5120 columns over up to 64 rows has two,
// one of 6144 columns four: 4096-wide with 8 key/value heads, or 2048-wide.  Requesting the later slots of q, k and v together too
// takes 0.3 - 0.6 us off the 17 - 20 of those, and adds 0.4 to the 14.2 of 4096 x 3 at 1K keys and 1 to the 22 - 30 of 8-bit rows.)
template <int F>
struct RowSums {
  float4 a[2][F / 4], b[2][F / 4];
  const float* src;
  int n;
  __device__ inline void load(const Partials& part, int64_t row, int col, int f0) {
    n = part.count(col);
    src = part.p + row * part.ld + col + f0;
#pragma unroll
    for (int p = 0; p < 2; ++p)
      if (p < n) {
#pragma unroll
        for (int i = 0; i < F / 4; ++i) {
          a[p][i] = *reinterpret_cast<const float4*>(src + p * part.stride + 4 * i);
          b[p][i] = *reinterpret_cast<const float4*>(src + p * part.stride + 64 + 4 * i);
        }
      }
  }
  __device__ inline void sum(const Partials& part, float (&lo)[F], float (&hi)[F]) const {
    auto add = [](float* s, const float4& v) { s[0] += v.x, s[1] += v.y, s[2] += v.z, s[3] += v.w; };
#pragma unroll
    for (int i = 0; i < F; ++i) lo[i] = hi[i] = 0.f;
#pragma unroll
    for (int p = 0; p < 2; ++p)
      if (p < n) {
#pragma unroll
        for (int i = 0; i < F / 4; ++i) add(lo + 4 * i, a[p][i]), add(hi + 4 * i, b[p][i]);
      }
    for (int p = 2; p < n; ++p) {
#pragma unroll
      for (int i = 0; i < F / 4; ++i) {
        add(lo + 4 * i, *reinterpret_cast<const float4*>(src + p * part.stride + 4 * i));
        add(hi + 4 * i, *reinterpret_cast<const float4*>(src + p * part.stride + 64 + 4 * i));
      }
    }
  }
};
// cos, sin of F rotary pairs
template <int F>
struct RopeRow {
  float4 cs[F / 2];
  __device__ inline void load(const float* cs_row, int f0) {
#pragma unroll
    for (int i = 0; i < F / 2; ++i) cs[i] = *reinterpret_cast<const float4*>(cs_row + 2 * f0 + 4 * i);
  }
  __device__ inline float cos(int i) const { return i & 1 ? cs[i >> 1].z : cs[i >> 1].x; }
  __device__ inline float sin(int i) const { return i & 1 ? cs[i >> 1].w : cs[i >> 1].y; }
  // Every product and rounding is written out: left to the compiler, which of a rotation's two products is rounded first, and
  // whether a binary16 result passes through fp32, differs from one instantiation to the next, and a node's K row with it.
  __device__ inline float low(float x, float y, int i) const { return fmaf(x, cos(i), -(y * sin(i))); }
  __device__ inline float high(float x, float y, int i) const { return fmaf(y, cos(i), x * sin(i)); }
  __device__ inline void rotate(float (&lo)[F], float (&hi)[F]) const {
#pragma unroll
    for (int i = 0; i < F; ++i) {
      const float x = lo[i], y = hi[i];
      lo[i] = low(x, y, i), hi[i] = high(x, y, i);
    }
  }
  // rotated pairs as E, two to a word.  (KEY: the upper features through fp32, as K rows have always had them.)
  template <typename E, bool KEY>
  __device__ inline void rotate_to(const float (&x)[F], const float (&y)[F], uint32_t (&lo)[F / 2], uint32_t (&hi)[F / 2]) const {
#pragma unroll
    for (int i = 0; i < F; i += 2) {
      lo[i / 2] = Elem16<E>::fma_pack2(x[i], cos(i), -(y[i] * sin(i)), x[i + 1], cos(i + 1), -(y[i + 1] * sin(i + 1)));
      if constexpr (KEY) {
        float h0 = high(x[i], y[i], i), h1 = high(x[i + 1], y[i + 1], i + 1);
        asm("" : "+v"(h0), "+v"(h1));
        hi[i / 2] = Elem16<E>::pack2(h0, h1);
      } else {
        hi[i / 2] = Elem16<E>::fma_pack2(y[i], cos(i), x[i] * sin(i), y[i + 1], cos(i + 1), x[i + 1] * sin(i + 1));
      }
    }
  }
};
// F elements, two to a word, to LDS (8 bytes at a time where F is 4)
template <int N>
__device__ inline void stage(uint8_t* dst, const uint32_t (&w)[N]) {
  if constexpr (N == 2) {
    *reinterpret_cast<uint2*>(dst) = uint2{w[0], w[1]};
  } else {
#pragma unroll
    for (int i = 0; i < N; i += 4) *reinterpret_cast<u32x4*>(dst + 4 * i) = u32x4{w[i], w[i + 1], w[i + 2], w[i + 3]};
  }
}

// qkv.p == NULL: q holds the rotated queries and the cache already holds the tree rows (separate RoPE kernel).
// qkv.p != NULL: the kernel starts from the QKV GEMM's partial sums: it reduces them, rotates q and k (RoPE,
// cos/sin table cs [row][64][2]), keeps q in LDS, and — if its key range reaches the tree slots — the tree's rows of K and V of
// its head too, from where they enter the product; one workgroup per key/value head also writes them into the cache.
// NU = 2: a workgroup carries all 64 queries (two groups of 32).  NU = 1: it carries 32 of them, the two halves of a
// (sequence, head, split) being two workgroups (blockIdx.z = 2 * sequence + half): half the accumulators, so two
// workgroups share a CU and twice as many loads are in flight per CU, at the price of K and V passing through the
// CU twice (the second time from L2: the halves are a multiple of 8 workgroups apart, i.e. on one XCD).
// TQ: nodes of the tree = queries of a sequence (64, or 15: one group of 32 of which the last 17 are padding that is
// never stored.  Six sequences of 40 .. 1500 keys x 32 heads take 30 us per layer; the portable kernel took 928 us
// for them).  Its softmax weights enter the product with V as the 16-bit terms of their fp32 values (WeightTerms, common.h): the
// portable kernel multiplies fp32 weights, and a tree is served with the same precision whichever of the two its shape takes.
// ONCE: no other workgroup reads this one's K and V blocks (it carries all queries of an ungrouped head), so they are loaded
// non-temporally: the stream then runs faster (as the weights', gemm_mfma.hip).  us per layer, plain / non-temporal: one sequence at
// 16K keys 65 / 59.6, 16 sequences of 256 .. 4096 keys 148 / 132,
// a step of 12 of 300 .. 4000 on the 15-node tree, 4 layers 1201 / 1173.  Where two halves share the blocks through L2 it costs (3
// sequences of 200 .. 2500 keys 31.2 / 34.9).
template <typename E, bool Q8, int NU, int TQ, bool ONCE>
__global__ void __launch_bounds__(256, NU == 1 ? 2 : 1)
    attn_tree_mfma_kernel(int tree, const E* __restrict__ q, const Partials qkv, const float* __restrict__ cs,
                          KvGeom g, E* __restrict__ kc, E* __restrict__ vc, int layer,
                          const int32_t* __restrict__ seq_len, int max_prefix, E* __restrict__ att_out,
                          float* __restrict__ part_o, float* __restrict__ part_ml, bool ordered) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  MDZ_STAMP(0);
  const TreeTables& t = c_trees[tree];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int qi = lane & 31, gh = lane >> 5;
  constexpr int kQW = 32 * NU;          // queries of this workgroup
  constexpr int kOPadN = kQW + 2;       // LDS row stride of the merge buffer (floats): conflict-free writes and reads
  const int split = blockIdx.x, n_splits = gridDim.x, h = blockIdx.y;
  constexpr int kHalves = TQ > kQW ? 2 : 1;  // workgroups that share a sequence's queries
  constexpr int kRows = TQ < kQW ? TQ : kQW;  // queries of this workgroup that exist
  constexpr bool kFp32Weights = TQ == 15;
  static_assert(!kFp32Weights || (NU == 1 && !Q8), "fp32 weights: one group of queries, 16-bit rows");
  const int b = ordered ? sequence_in_order(seq_len, gridDim.z / kHalves, blockIdx.z / kHalves) : blockIdx.z / kHalves;
  const int q0 = (blockIdx.z % kHalves) * 32;  // first query of this workgroup
  const int hk = h / g.group;  // the key/value head that query head h reads (grouped-query attention)
  const int d = q_heads(g) * kHD, dkv = g.n_heads * kHD;
  const int S = min(max(seq_len[b], 0), max_prefix);
  const int n_slots = S + TQ;
  const int nb = (n_slots + 31) >> 5;
  int blk_begin, blk_end;
  if (qkv.p != nullptr && n_splits > 1) {  // last split: every block with a tree slot; the others: prefix-only blocks
    // (With one or two prefix splits the tree split also takes what it has time for at the end of the prefix: its prologue is
    // worth about 24 blocks of a prefix split, 32 with 8-bit rows.  3 sequences of 200 .. 2500 keys, two splits: 37.8 -> 31.6 us
    // per layer; with five to seven prefix splits nothing is gained: 29.3 / 28.9 us at 7K keys of 8 bits, 65.3 / 66.6 at 16K of 16 bits.
    // us per step of 4 layers with 10 / 16 / 24 / 32 blocks: 3 sequences 1020 / 1016 / 1010 / 1016, 4 of 300 .. 3400 1183 / 1188 / 1193 / 1206, one of
    // 2000 662 / 662 / 657 / 655, 4 of 200 .. 2500 with 8-bit rows 1135 / 1131 / 1125 / 1114.)
    constexpr int kTreeCost = Q8 ? 32 : 24;
    const int ps = n_splits - 1, all = S >> 5;
    const int extra = ps == 1 ? max((all - kTreeCost) / 2, 0) : ps == 2 ? max((all - 2 * kTreeCost) / 3, 0) : 0, pb = all - extra;
    blk_begin = split == ps ? pb : (int)((int64_t)split * pb / ps);
    blk_end = split == ps ? nb : (int)((int64_t)(split + 1) * pb / ps);
  } else {
    blk_begin = (int)((int64_t)split * nb / n_splits);
    blk_end = (int)((int64_t)(split + 1) * nb / n_splits);
  }

  // 16-bit rows: block blk, unit i at kp[blk*512 + i*64].  8-bit rows: a block is 264 16-byte pieces: unit i at
  // kp[blk*264 + i*64], the four scales of keys 8j + 4gh .. +3 at ks_p[blk*264 + 2j]
  constexpr int kBlkPieces = Q8 ? kKv8BlockBytes / 16 : 512;
  const u32x4* kp;
  const u32x4* vp;
  const u32x4* ks_p = nullptr;
  const u32x4* vs_p = nullptr;
  if constexpr (Q8) {
    const int64_t hb = kv8_head_base(g, layer, b, hk);
    const u32x4* k0 = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(kc) + hb);
    const u32x4* v0 = reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(vc) + hb);
    kp = k0 + lane, vp = v0 + lane;
    ks_p = k0 + 256 + gh, vs_p = v0 + 256 + gh;
  } else {
    const int64_t head_base = kv_head_base(g, layer, b, hk);
    kp = reinterpret_cast<const u32x4*>(kc + head_base) + lane;
    vp = reinterpret_cast<const u32x4*>(vc + head_base) + lane;
  }

  // K and V are both double buffered one block ahead of the block being multiplied, and every load is
  // unconditional (past the wave's last block it repeats that block and the result is not used): the wait counters
  // are in-order, so a wave then keeps a whole block (16 KiB of 16-bit rows) in flight while it works on the
  // previous one, which is what the HBM latency asks for at one wave per SIMD.
  u32x4 kb[2][8], vb[2][8];
  auto unit = [](const u32x4* p) { return ONCE ? __builtin_nontemporal_load(p) : *p; };
  auto load_kv = [&](int blk, u32x4 (&kd)[8], u32x4 (&vd)[8]) {  // 8-bit rows: [0..3] codes, [4..7] the lane's 16 scales
#pragma unroll
    for (int i = 0; i < 8; ++i)
      kd[i] = (Q8 && i >= 4) ? ks_p[(int64_t)blk * kBlkPieces + 2 * (i - 4)] : unit(kp + (int64_t)blk * kBlkPieces + i * 64);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      vd[i] = (Q8 && i >= 4) ? vs_p[(int64_t)blk * kBlkPieces + 2 * (i - 4)] : unit(vp + (int64_t)blk * kBlkPieces + i * 64);
  };
  // this wave's blocks: blk_begin + wave, + 4, ... ; two per trip so that the buffers alternate statically
  const int n_mine = blk_begin + wave < blk_end ? (blk_end - blk_begin - wave + 3) >> 2 : 0;
  const int first = blk_begin + wave, last = first + 4 * (n_mine - 1);
  // Fused: does this workgroup's range reach the tree slots?  Its blocks there take the tree's K and V rows from LDS.
  const bool has_tree = qkv.p != nullptr && split == n_splits - 1;
  // Q tile of this head -> LDS (rows padded by 16 B: the 16 B-per-lane operand reads below are bank-conflict
  // free), then, where the range reaches the tree slots, the tree's K and V rows (16-bit, or 128 codes and a scale).  The region is
  // reused by the wave merge after the key loop.
  uint8_t* q_lds = reinterpret_cast<uint8_t*>(lds);
  uint8_t* k_lds = q_lds + kQW * kQRow;
  uint8_t* v_lds = k_lds + TQ * kQRow;
  if (qkv.p == nullptr) {
#pragma unroll
    for (int i = 0; i < 2 * NU; ++i) {
      int idx = threadIdx.x + i * 256;
      int row = idx >> 4, col = idx & 15;
      *reinterpret_cast<u32x4*>(q_lds + row * kQRow + col * 16) =
          *reinterpret_cast<const u32x4*>(q + (int64_t)(b * TQ + q0 + min(row, kRows - 1)) * d + h * kHD + col * 8);
    }
    if (n_mine > 0) load_kv(first, kb[0], vb[0]);
  } else {
    // Bound by its round trips to memory, which cost 3 - 4 us each while other workgroups stream: the loads of the first two slots
    // of q, k and v and of their rotations are requested before the first is used, and nothing is read back from the cache.  One
    // tree of 64 nodes, two slots: 7.8 us with the matrices one after the other, slot by slot, and the rows through the cache.
    // (us per layer, that way / this way: 3 x 4096 columns at 1K keys 16.7 / 14.2, four slots 19.3 / 17.8.)
    // Thread (row, seg): F features from F * seg on, and their partners, of a row; 256 threads cover the rows.
    constexpr int kKvThreads = TQ == 15 ? 16 : 4, kKvF = 64 / kKvThreads;
    constexpr int kQThreads = TQ == 15 ? 16 : 256 / kQW, kQF = 64 / kQThreads;
    const int kv_row = min((int)threadIdx.x / kKvThreads, TQ - 1), kv_f0 = (threadIdx.x % kKvThreads) * kKvF;
    const int q_row = threadIdx.x / kQThreads, q_f0 = (threadIdx.x % kQThreads) * kQF;
    const int64_t grow_kv = (int64_t)b * TQ + kv_row, grow_q = (int64_t)b * TQ + q0 + min(q_row, kRows - 1);
    RowSums<kQF> qs;
    RopeRow<kQF> q_rope;
    auto stage_q = [&]() {
      float x[kQF], y[kQF];
      uint32_t lo[kQF / 2], hi[kQF / 2];
      qs.sum(qkv, x, y);
      q_rope.template rotate_to<E, false>(x, y, lo, hi);
      uint8_t* dst = q_lds + q_row * kQRow + 2 * q_f0;
      stage(dst, lo);
      stage(dst + 128, hi);
      if constexpr (TQ == 15) {  // the padding columns of the operand: copies
        stage(dst + 16 * kQRow, lo);
        stage(dst + 16 * kQRow + 128, hi);
      }
    };
    if (has_tree) {
      RowSums<kKvF> ks, vs;
      RopeRow<kKvF> k_rope;
      ks.load(qkv, grow_kv, d + hk * kHD, kv_f0);
      k_rope.load(cs + grow_kv * kHD, kv_f0);
      qs.load(qkv, grow_q, h * kHD, q_f0);
      q_rope.load(cs + grow_q * kHD, q_f0);
      vs.load(qkv, grow_kv, d + dkv + hk * kHD, kv_f0);
      __builtin_amdgcn_sched_barrier(0);
      uint8_t* k_dst = k_lds + kv_row * kQRow;
      uint8_t* v_dst = v_lds + kv_row * kQRow;
      // an 8-bit row: its scale, from the largest magnitude over its 4 threads, and the codes of this thread's 2 x 16 features
      auto stage_codes = [&](uint8_t* dst, const float (&lo)[kKvF], const float (&hi)[kKvF]) {
        float am = 0.f;
#pragma unroll
        for (int i = 0; i < kKvF; ++i) am = fmaxf(am, fmaxf(fabsf(lo[i]), fabsf(hi[i])));
        am = fmaxf(am, __shfl_xor(am, 1, 64));
        am = fmaxf(am, __shfl_xor(am, 2, 64));
        const float sc = kv8_scale_of(am);
#pragma unroll
        for (int i = 0; i < kKvF; i += 4) {
          *reinterpret_cast<uint32_t*>(dst + kv_f0 + i) = kv8_pack4(lo[i], lo[i + 1], lo[i + 2], lo[i + 3], sc);
          *reinterpret_cast<uint32_t*>(dst + 64 + kv_f0 + i) = kv8_pack4(hi[i], hi[i + 1], hi[i + 2], hi[i + 3], sc);
        }
        if (kv_f0 == 0) *reinterpret_cast<float*>(dst + 128) = sc;
      };
      auto stage_words = [&](uint8_t* dst, const uint32_t (&lo)[kKvF / 2], const uint32_t (&hi)[kKvF / 2]) {
        stage(dst + 2 * kv_f0, lo);
        stage(dst + 128 + 2 * kv_f0, hi);
      };
      {
        float x[kKvF], y[kKvF];
        ks.sum(qkv, x, y);
        if constexpr (Q8) {
          k_rope.rotate(x, y);
          stage_codes(k_dst, x, y);
        } else {
          uint32_t lo[kKvF / 2], hi[kKvF / 2];
          k_rope.template rotate_to<E, true>(x, y, lo, hi);
          stage_words(k_dst, lo, hi);
        }
      }
      stage_q();
      {
        float x[kKvF], y[kKvF];
        vs.sum(qkv, x, y);
        if constexpr (Q8) {
          stage_codes(v_dst, x, y);
        } else {
          uint32_t lo[kKvF / 2], hi[kKvF / 2];
#pragma unroll
          for (int i = 0; i < kKvF; i += 2) lo[i / 2] = Elem16<E>::pack2(x[i], x[i + 1]), hi[i / 2] = Elem16<E>::pack2(y[i], y[i + 1]);
          stage_words(v_dst, lo, hi);
        }
      }
      if (n_mine > 0) load_kv(first, kb[0], vb[0]);
    } else {
      // Prefix splits request their first block first: the loads behind it then wait no longer than this one takes.
      // (not for 8-bit rows with 64 queries: that variant has no registers to hold the block meanwhile)
      if (!(Q8 && NU == 2) && n_mine > 0) load_kv(first, kb[0], vb[0]);
      qs.load(qkv, grow_q, h * kHD, q_f0);
      q_rope.load(cs + grow_q * kHD, q_f0);
      stage_q();
      if (Q8 && NU == 2 && n_mine > 0) load_kv(first, kb[0], vb[0]);
    }
  }
  MDZ_STAMP(1);
  __syncthreads();  // Q tile and tree rows complete
  MDZ_STAMP(2);
  // B operand of scores^T: lane holds query 32u + qi, features 16ks + 8gh .. +7
  const uint8_t* qfrag = q_lds + qi * kQRow + gh * 16;
  uint64_t mq[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) mq[u] = t.anc_mask[min(q0 + 32 * u + qi, TQ - 1)];
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)kHD);

  float m_run[NU], l_run[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) m_run[u] = -INFINITY, l_run[u] = 0.f;
  f32x16 o[4][NU];
#pragma unroll
  for (int tt = 0; tt < 4; ++tt)
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[tt][u][r] = 0.f;

  auto process = [&](int blk, const u32x4 (&kd)[8], const u32x4 (&vd)[8], auto masked) {
    // Compiler barrier: keeps the (loop-invariant) Q operand reads inside the loop, i.e. in LDS rather
    // than in 64 registers per lane that this kernel does not have to spare.
    asm volatile("" ::: "memory");
    f32x16 sc[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[u][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const u32x4 ka = Q8 ? fp8x8_to_elem<E>(kd[ks >> 1], ks & 1) : kd[ks];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const u32x4 qv = *reinterpret_cast<const u32x4*>(qfrag + u * 32 * kQRow + ks * 32);
        sc[u] = Elem16<E>::mfma(ka, qv, sc[u]);
      }
    }
    // Visibility of this block's 32 keys for the lane's query, as one 32-bit word: prefix keys are
    // visible, a tree key S+j is visible iff bit j of the query's ancestor mask is set, keys beyond the
    // tree are not.  rel0 (wave-uniform) = offset of the block's first key from the tree's first slot.
    const int rel0 = blk * 32 - S;
    constexpr bool need_mask = decltype(masked)::value;  // the block reaches past the prefix
    float alpha[NU];
    u32x4 pf[NU][2];
    float weight[16];  // (fp32 weights: NU is 1)
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      float bmax = -INFINITY;
      // register r is key 8*(r/4) + 4*gh + r%4 of the block; its scale is component r%4 of scale piece r/4
      if constexpr (need_mask) {  // only the (at most three) blocks that hold tree slots pay for the mask
        const uint32_t pre = rel0 >= 0 ? 0u : (0xFFFFFFFFu >> (32 + rel0));          // keys below S (rel0 in [-31,-1])
        const uint64_t tr = rel0 >= 0 ? (mq[u] >> rel0) : (mq[u] << (-rel0));        // rel0 in [-31, 63]
        const uint32_t vis = (pre | (uint32_t)tr) >> (4 * gh);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float s = sc[u][r] * (Q8 ? __uint_as_float(kd[4 + (r >> 2)][r & 3]) * scale_log2 : scale_log2);
          s = ((vis >> (8 * (r >> 2) + (r & 3))) & 1u) ? s : -INFINITY;
          sc[u][r] = s;
          bmax = fmaxf(bmax, s);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float s = sc[u][r] * (Q8 ? __uint_as_float(kd[4 + (r >> 2)][r & 3]) * scale_log2 : scale_log2);
          sc[u][r] = s;
          bmax = fmaxf(bmax, s);
        }
      }
      bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));
      // The running reference m_run only has to keep exp2(s - m_run) in range, it need not be the maximum: it is
      // moved (and the accumulators rescaled: 128 registers through the vector ALU) only when a block's maximum
      // exceeds it by more than 2^kLazyLog2, so probabilities stay below 2^kLazyLog2 and, in a long prefix, almost
      // no block rescales.  o, l and m stay consistent, so the merges below need no change.
      // (fp32 weights: always the maximum, so that they are at most 1.)
      const float m_new = bmax > m_run[u] + (kFp32Weights ? 0.f : kLazyLog2) ? bmax : m_run[u];
      const float m_safe = m_new == -INFINITY ? 0.f : m_new;
      alpha[u] = m_new == m_run[u] ? 1.f : fast_exp2(m_run[u] - m_safe);
      float sum = 0.f;
      uint32_t pk[8];
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        float p0 = fast_exp2(sc[u][r] - m_safe), p1 = fast_exp2(sc[u][r + 1] - m_safe);
        if constexpr (kFp32Weights) {
          p0 *= WeightTerms<E>::kScale, p1 *= WeightTerms<E>::kScale;
          weight[r] = p0, weight[r + 1] = p1;
          sum += p0 + p1;
          continue;
        }
        sum += p0 + p1;
        if constexpr (Q8) p0 *= __uint_as_float(vd[4 + (r >> 2)][r & 3]), p1 *= __uint_as_float(vd[4 + (r >> 2)][(r & 3) + 1]);
        pk[r >> 1] = Elem16<E>::pack2(p0, p1);
      }
      l_run[u] = l_run[u] * alpha[u] + sum;
      m_run[u] = m_new;
      pf[u][0] = u32x4{pk[0], pk[1], pk[2], pk[3]};
      pf[u][1] = u32x4{pk[4], pk[5], pk[6], pk[7]};
    }
    if (__any(alpha[0] != 1.f || alpha[NU - 1] != 1.f)) {
#pragma unroll
      for (int tt = 0; tt < 4; ++tt)
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[tt][u][r] *= alpha[u];
    }
    if constexpr (kFp32Weights) {
#pragma unroll
      for (int i = 0; i < WeightTerms<E>::kTerms; ++i) {
        u32x4 term[2];
        next_weight_term<E>(weight, term);
#pragma unroll
        for (int tt = 0; tt < 4; ++tt)
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2) o[tt][0] = Elem16<E>::mfma(vd[tt * 2 + s2], term[s2], o[tt][0]);
      }
      return;
    }
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const u32x4 va = Q8 ? fp8x8_to_elem<E>(vd[tt], s2) : vd[tt * 2 + s2];
#pragma unroll
        for (int u = 0; u < NU; ++u) o[tt][u] = Elem16<E>::mfma(va, pf[u][s2], o[tt][u]);
      }
  };

  // Puts the tree's rows of block blk, staged in LDS, into its units (what the cache holds there is not yet written).
  auto put_tree = [&](int blk, u32x4 (&kd)[8], u32x4 (&vd)[8]) {
    const int n0 = blk * 32 - S;  // node of the block's first key; nodes outside [0, TQ) stay as loaded
    const bool mine = (unsigned)(n0 + qi) < (unsigned)TQ;
    const uint8_t* krow = k_lds + (mine ? n0 + qi : 0) * kQRow;
    const uint8_t* vcol = v_lds + (Q8 ? qi : 2 * qi);
    auto node = [&](int key) { return n0 + key + 4 * gh; };  // key: 8 * j + c, c < 4, of the half-wave's numbering
    auto in_tree = [&](int key) { return (unsigned)node(key) < (unsigned)TQ; };
    auto row_of = [&](int key) { return min(max(node(key), 0), TQ - 1) * kQRow; };
    if constexpr (Q8) {
      if (mine) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint2 lo = *reinterpret_cast<const uint2*>(krow + 32 * j + 8 * gh), hi = *reinterpret_cast<const uint2*>(krow + 32 * j + 16 + 8 * gh);
          kd[j] = u32x4{lo.x, lo.y, hi.x, hi.y};
        }
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)  // keys 8 j + 4 gh + c: byte 4 (j % 2) + c of V's word pair j / 2, component c of scale piece j
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          __builtin_amdgcn_sched_barrier(0);
          const int key = 8 * j + c, row = row_of(key);
          const bool in = in_tree(key);
          const uint32_t ksc = *reinterpret_cast<const uint32_t*>(k_lds + row + 128), vsc = *reinterpret_cast<const uint32_t*>(v_lds + row + 128);
          kd[4 + j][c] = in ? ksc : kd[4 + j][c];
          vd[4 + j][c] = in ? vsc : vd[4 + j][c];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const uint32_t code = vcol[row + 32 * t];
            vd[t][j] = in ? (vd[t][j] & ~(0xFFu << (8 * c))) | code << (8 * c) : vd[t][j];
          }
        }
    } else {
      if (mine) {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kd[ks] = *reinterpret_cast<const u32x4*>(krow + 32 * ks + 16 * gh);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j)  // keys 8 j + 4 gh + c: element 4 (j % 2) + c of unit 2 t + j / 2
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          __builtin_amdgcn_sched_barrier(0);
          const int key = 8 * j + c, row = row_of(key), w = 2 * (j & 1) + (c >> 1);
          const bool in = in_tree(key);
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const uint32_t v = *reinterpret_cast<const uint16_t*>(vcol + row + 64 * t), old = vd[2 * t + (j >> 1)][w];
            vd[2 * t + (j >> 1)][w] = in ? (c & 1 ? (old & 0xFFFFu) | v << 16 : (old & 0xFFFF0000u) | v) : old;
          }
        }
    }
  };
  // Stores the tree's rows of block blk and nothing else: other slots of the block may be written from another stream meanwhile.
  auto write_tree = [&](int blk, const u32x4 (&kd)[8], const u32x4 (&vd)[8]) {
    u32x4* kw = const_cast<u32x4*>(kp) + (int64_t)blk * kBlkPieces;
    u32x4* vw = const_cast<u32x4*>(vp) + (int64_t)blk * kBlkPieces;
    const int n0 = blk * 32 - S;
    const bool mine = (unsigned)(n0 + qi) < (unsigned)TQ;
    if (mine) {
#pragma unroll
      for (int i = 0; i < (Q8 ? 4 : 8); ++i) kw[i * 64] = kd[i];
    }
    if (n0 >= 0 && n0 + 32 <= TQ) {  // every key of the block is a node
#pragma unroll
      for (int i = 0; i < (Q8 ? 4 : 8); ++i) vw[i * 64] = vd[i];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // the lane's keys 8 j + 4 gh .. + 3 lie together, in word j of a unit or in a pair of words
        const int node = n0 + 8 * j + 4 * gh;
        if (node >= 0 && node + 4 <= TQ) {
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            if constexpr (Q8) {
              reinterpret_cast<uint32_t*>(vw + t * 64)[j] = vd[t][j];
            } else {
              const u32x4 v = vd[2 * t + (j >> 1)];
              reinterpret_cast<uint2*>(vw + (2 * t + (j >> 1)) * 64)[j & 1] = j & 1 ? uint2{v.z, v.w} : uint2{v.x, v.y};
            }
          }
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            if ((unsigned)(node + c) < (unsigned)TQ) {
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                if constexpr (Q8)
                  reinterpret_cast<uint8_t*>(vw + t * 64)[4 * j + c] = (uint8_t)(vd[t][j] >> (8 * c));
                else
                  reinterpret_cast<uint16_t*>(vw + (2 * t + (j >> 1)) * 64)[4 * (j & 1) + c] =
                      (uint16_t)(vd[2 * t + (j >> 1)][2 * (j & 1) + (c >> 1)] >> (16 * (c & 1)));
              }
            }
        }
      }
    }
    if constexpr (Q8) {  // scales: lane gh = 0 of a key
      if (mine && gh == 0) {
        const int row = (n0 + qi) * kQRow;
        reinterpret_cast<uint32_t*>(kw - lane + 256)[qi] = *reinterpret_cast<const uint32_t*>(k_lds + row + 128);
        reinterpret_cast<uint32_t*>(vw - lane + 256)[qi] = *reinterpret_cast<const uint32_t*>(v_lds + row + 128);
      }
    }
  };

  // The blocks wholly in the prefix, then the wave's block with tree slots, if it has one (three at most, so one per wave).
  if (n_mine > 0) {
    const bool tail = last * 32 + 32 > S;
    const int n_pre = n_mine - (tail ? 1 : 0);
    for (int it = 0; it < n_pre; it += 2) {
      const int blk = first + 4 * it;
      load_kv(min(blk + 4, last), kb[1], vb[1]);
      __builtin_amdgcn_sched_barrier(0);
      process(blk, kb[0], vb[0], std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
      load_kv(min(blk + 8, last), kb[0], vb[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (it + 1 < n_pre) process(blk + 4, kb[1], vb[1], std::false_type{});
      __builtin_amdgcn_sched_barrier(0);
    }
    if (tail) {  // (block `last` is in the first buffer: the loop's last load repeats it)
      if (has_tree) {
        put_tree(last, kb[0], vb[0]);
        // one of the workgroups that hold these rows writes them
        if (h % g.group == 0 && q0 == 0) write_tree(last, kb[0], vb[0]);
      }
      process(last, kb[0], vb[0], std::true_type{});
    }
  }

  MDZ_STAMP(3);
  // ---- merge the four waves through LDS (fixed order) ------------------------------------------
  __syncthreads();  // every wave is done reading the Q tile that the merge buffer overlays
  float* o_lds = lds;                             // [4][kHD][kOPadN]
  float* m_lds = lds + 4 * kHD * kOPadN;          // [4][kQW]
  float* l_lds = m_lds + 4 * kQW;                 // [4][kQW]
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    float l_tot = l_run[u] + __shfl_xor(l_run[u], 32, 64);
    if (gh == 0) {
      m_lds[wave * kQW + 32 * u + qi] = m_run[u];
      l_lds[wave * kQW + 32 * u + qi] = l_tot;
    }
#pragma unroll
    for (int tt = 0; tt < 4; ++tt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        int hd = 32 * tt + 8 * (r >> 2) + 4 * gh + (r & 3);
        o_lds[(wave * kHD + hd) * kOPadN + 32 * u + qi] = o[tt][u][r];
      }
  }
  __syncthreads();
  // kTPQ threads per query; thread (qq = t / kTPQ, s = t % kTPQ) merges features 16*jj + kEW*s + e (jj < 8, e < kEW)
  constexpr int kTPQ = 256 / kQW, kEW = 16 / kTPQ;
  const int qq = threadIdx.x / kTPQ, s4 = (threadIdx.x % kTPQ) * kEW;
  float mw[4], M = -INFINITY;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    mw[w] = m_lds[w * kQW + qq];
    M = fmaxf(M, mw[w]);
  }
  const float M_safe = M == -INFINITY ? 0.f : M;
  float L = 0.f, wt[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    wt[w] = fast_exp2(mw[w] - M_safe);
    L += wt[w] * l_lds[w * kQW + qq];
  }
  float acc[8 * kEW];
#pragma unroll
  for (int j = 0; j < 8 * kEW; ++j) {
    const int f = 16 * (j / kEW) + s4 + (j % kEW);
    float a = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) a += wt[w] * o_lds[(w * kHD + f) * kOPadN + qq];
    acc[j] = a;
  }
  const int q_out = q0 + qq;  // the query's row among those of its sequence
  if (kRows < kQW && qq >= kRows) return;
  if (n_splits == 1) {
    const float inv = 1.0f / L;
    E* dst = att_out + (int64_t)(b * TQ + q_out) * d + h * kHD + s4;
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
      if constexpr (kEW == 4)
        *reinterpret_cast<uint2*>(dst + 16 * jj) = uint2{Elem16<E>::pack2(acc[4 * jj] * inv, acc[4 * jj + 1] * inv),
                                                         Elem16<E>::pack2(acc[4 * jj + 2] * inv, acc[4 * jj + 3] * inv)};
      else
        *reinterpret_cast<uint32_t*>(dst + 16 * jj) = Elem16<E>::pack2(acc[2 * jj] * inv, acc[2 * jj + 1] * inv);
    }
  } else {
    const int64_t pidx = ((int64_t)(b * q_heads(g) + h) * n_splits + split);
    float* po = part_o + (pidx * TQ + q_out) * kHD + s4;
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
      if constexpr (kEW == 4)
        *reinterpret_cast<float4*>(po + 16 * jj) = float4{acc[4 * jj], acc[4 * jj + 1], acc[4 * jj + 2], acc[4 * jj + 3]};
      else
        *reinterpret_cast<float2*>(po + 16 * jj) = float2{acc[2 * jj], acc[2 * jj + 1]};
    }
    if (threadIdx.x % kTPQ == 0) {
      part_ml[(pidx * 2 + 0) * TQ + q_out] = M;
      part_ml[(pidx * 2 + 1) * TQ + q_out] = L;
    }
  }
  MDZ_STAMP(4);
}

// Merges the key-splits of 16 queries of one (sequence, head): fixed order, exact same weighting rule as above.
// Thread (q = t/16, c = t%16) owns features 8c .. 8c+7 of query 16*blockIdx.z + q.
template <typename E, int TQ>
__global__ void __launch_bounds__(256)
    attn_combine_kernel(int n_heads, int n_splits, const float* __restrict__ part_o, const float* __restrict__ part_ml,
                        E* __restrict__ att_out) {
  const int h = blockIdx.x, b = blockIdx.y;
  const int d = n_heads * kHD;
  const int qq = blockIdx.z * 16 + (threadIdx.x >> 4), f0 = (threadIdx.x & 15) * 8;
  if (TQ % 16 != 0 && qq >= TQ) return;
  const int64_t p0 = (int64_t)(b * n_heads + h) * n_splits;
  float M = -INFINITY;
  float L = 0.f;
  float acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = 0.f;
  // Splits are taken eight at a time: the loads of a group are all requested before the first is used, so a merge of
  // many splits costs one memory round trip per eight, not one per split.  The weights refer to the running maximum
  // of the groups seen so far (the sums are rescaled when a later group raises it), in a fixed order.
  constexpr int kTogether = 8;
  for (int s0 = 0; s0 < n_splits; s0 += kTogether) {
    float ms[kTogether], ls[kTogether];
    float4 v0[kTogether], v1[kTogether];
#pragma unroll
    for (int s = 0; s < kTogether; ++s)
      if (s0 + s < n_splits) {
        ms[s] = part_ml[((p0 + s0 + s) * 2 + 0) * TQ + qq];
        ls[s] = part_ml[((p0 + s0 + s) * 2 + 1) * TQ + qq];
        const float4* po = reinterpret_cast<const float4*>(part_o + ((p0 + s0 + s) * TQ + qq) * kHD + f0);
        v0[s] = po[0], v1[s] = po[1];
      }
    float Mg = M;
#pragma unroll
    for (int s = 0; s < kTogether; ++s)
      if (s0 + s < n_splits) Mg = fmaxf(Mg, ms[s]);
    if (Mg != M) {  // (first group: M = -inf and the sums are zero)
      const float r = M == -INFINITY ? 0.f : fast_exp2(M - Mg);
      L *= r;
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[j] *= r;
      M = Mg;
    }
#pragma unroll
    for (int s = 0; s < kTogether; ++s)
      if (s0 + s < n_splits) {
        const float w = ms[s] == -INFINITY ? 0.f : fast_exp2(ms[s] - M);  // (an empty split, possibly before any other: M = -inf)
        L += w * ls[s];
        acc[0] += w * v0[s].x, acc[1] += w * v0[s].y, acc[2] += w * v0[s].z, acc[3] += w * v0[s].w;
        acc[4] += w * v1[s].x, acc[5] += w * v1[s].y, acc[6] += w * v1[s].z, acc[7] += w * v1[s].w;
      }
  }
  const float inv = 1.0f / L;
  uint32_t pk[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) pk[j] = Elem16<E>::pack2(acc[2 * j] * inv, acc[2 * j + 1] * inv);
  *reinterpret_cast<u32x4*>(att_out + (int64_t)(b * TQ + qq) * d + h * kHD + f0) = u32x4{pk[0], pk[1], pk[2], pk[3]};
}

bool attn_mfma_supported(int dtype, int tree, const KvGeom& g) {
  return is_16bit(dtype) && g.tiled && g.head_dim == kHD &&
         (host_tree(tree)->T == 64 || (host_tree(tree)->T == 15 && !g.quant));
}

// Key-splits of a launch with 32 queries per workgroup (see attn_plan)
static int halves_splits(int B, int pairs, int max_prefix, bool grouped) {
  const int by_len = 1 + (int)sqrtf((float)(max_prefix >> 5) / 8.0f), cus = num_cus();
  if (B == 1 && grouped && by_len * pairs >= cus) return cus / pairs;
  const int most = B == 1 || max_prefix < 1536 ? cus / (2 * pairs) : max_prefix < 2048 ? cus * 9 / 8 / (2 * pairs) : cus / pairs;
  return most < 1 ? 1 : by_len < most ? by_len : most;
}

// Key-splits that fill the CUs with a workgroup each: ungrouped heads four fifths of them (see attn_plan)
static int full_splits(const KvGeom& g, int B, int pairs) {
  return g.group > 1 ? num_cus() / pairs : num_cus() * 4 / 5 / pairs + (B > 1);
}

// Queries per workgroup and key-splits per (sequence, head) of a launch.
struct AttnPlan {
  bool halves;  // 32 queries per workgroup (two fit a CU), else 64
  int splits;
  bool ordered;  // the longest sequences first
};

// fused: the kernel starts from the QKV partial sums, so one split is the tree split and the rest share the prefix.  Every further split
// costs about a microsecond per layer (its reduce of the Q partial sums, its share of the merge) and saves the blocks it takes off the
// others, so the best count grows with the square root of the prefix, up to a workgroup on every CU: 32 queries per workgroup (B = 1: one per
// CU; a CU with two beside CUs with one is the last to end), 64 queries: four fifths of the CUs (at all of them, with 8 splits, every split of
// a head lies on an XCD of its own, and the tree splits' XCD idles).  With 32 queries K and V pass through the CUs twice, which costs more than
// the shorter chain of a workgroup saves once they are many.  us, steps of 4 layers, 64 nodes (h: 32 queries; s: splits):
//   32 heads, one sequence: 1024 keys h s2 617, h s3 614, h s4 618; 4000 keys s4 691, s6 679, h s4 657; 5500 s6 687, h s4 687; 7000 s6 701, s8 711,
//     h s4 711; 16384 s6 800, s7 803, s8 818, h s4 844.  16 heads: 4000 s4 405, h s4 353; 7000 s6 413, s12 393, h s4 370, h s6 355; 10000 s8 419,
//     h s8 398; 14000 s8 441, s12 422, h s8 425.  40 heads: 4000 s4 725, h s3 707, h s4 728; 7000 s5 753, s6 758, h s3 754; 14000 s5 832, s6 853.
//   8-bit rows, 32 heads: 7000 h s6 665, h s4 659, s8 670; 10000 h s7 705, h s4 696, s8 703; 14000 h s4 732, s6 756, s8 729.
//   four query heads to a key/value head (their blocks come from L2, the better for a workgroup per CU, i.e. a split on each XCD): 4000 s4 728, h s4 677; 7000 s6
//     719, h s4 694; 10 layers: 8000 s8 1316, h s4 1313, h s8 1304, 11500 s8 1368, h s4 1390, h s8 1367, 13500 s8 1396, h s4 1440, h s8 1406; 8-bit rows 13000 s8 1417,
//     h s4 1367, h s8 1351, 20000 s8 1531, h s4 1494, h s8 1455.
//   several sequences (n / 8 .. n keys; the longest is the last to end, so long ones take twice the splits): 2 at 1500 h s2 788, h s3 802; 4000 s4 864,
//     h s4 853; 8000 s3 922, s4 923, h s4 926; 3 at 1500 h s1 892, h s2 901 (3 x 16 heads, 16 layers, 1100 h s2
//     1520, h s3 1519, 1700 h s2 1573, h s3 1556); 2500 h s1 931, h s2 922; 8000 s2 1091, s3 1060; 4 at 600 h s1 1002, h s2 1025.
//   8-bit rows of several sequences are converted by more CUs with 32 queries, whatever the length (2 layers, h / 64 queries): 2 at 14000 374 / 420, 3 at
//     11000 435 / 498, 4 at 8000 482 / 513, 5 at 6000 557 / 631, 22000 782 / 1010, 8 at 8000 748 / 796, of equal length within 1 % or better.
//   more pairs than half the CUs, hence one split (3 layers, h / 64 queries, lengths n / 8 .. n and n / 2 .. n): 5 x 32 heads at 2500 739 / 741 and 771 / 751,
//     6 at 3400 814 / 813 and 869 / 835, 7 at 3200 (4 layers) 1316 / 1263 and 1365 / 1291, 9 x 16 at 3000 500 / 500 and 539 / 501, 11 at 3000 598 / 546 and
//     604 / 553, 4 x 40 at 2500 866 / 840 and 886 / 848 (32 queries are ahead by at most 1 %, where five or six lengths spread from n / 20);
//     grouped heads (2 layers): 5 at 3000 503 / 521 and 523 / 526, 8 at 3000 627 / 632 and 649 / 654.
//   15 nodes, one sequence: 1000 s3 573, s5 568; 4000 s4 609, s6 595; 8000 s4 664, s6 632; two 2000 s3 613, s4 604, s6 614; 8000 s4 688, s6 673; three 2000 s2
//     650, s4 644; 8000 s2 779, s4 759, s5 780; four 2000 s2 666, s4 678; six 2000 s1 784, s2 802.  10 layers, grouped heads, one: 14000 s6 1277, s7 1283, s8 1170 (two
//     at 4500 s6 1134, s8 1095, one at 7000 s6 1129, s8 1081: left, the count is of the length); 32 heads 14000 s6 1318, s8 1365.  16 layers of 16 heads: one 10000 s6 1180,
//     s7 1138, 14000 s6 1310, s8 1220; two 14000 s6 1395, s7 1335; three 4500 s4 1287, s5 1244, s6 1279; four 4500 s4 1366, s6 1418; five 4500 s3 1496, s4 1519 (2100 1338,
//     1336); six 4500 s2 1649, s4 1617.  8 layers of 40 heads: two 4500 s3 1248, s4 1263.
static AttnPlan attn_plan(int T, const KvGeom& g, int B, int max_prefix, bool fused) {
  const int pairs = B * q_heads(g), cus = num_cus(), nb = max_prefix >> 5;
  const int by_len = 1 + (int)sqrtf((float)nb / 8.0f);
  AttnPlan p{true, 1, false};
  auto at_most = [](int a, int b) { return a < b ? a : b; };
  auto at_least = [](int a, int b) { return a > b ? a : b; };
  if (T == 64) {
    const double through = (double)pairs * max_prefix * (g.quant ? 264 : 512);  // bytes of K and V that a launch takes through the CUs once
    p.halves = pairs <= cus && ((g.quant && B > 1) || (g.group > 1 && max_prefix < 3584) ||
                                through <= (B == 1 ? 96e6 : 160e6) * (g.group > 1 ? (B == 1 && !g.quant ? 2.0 : 2.5) : g.quant ? 1.3 : 1.0));
  }
  if (!fused) {
    const int most = (max_prefix + T + 31) / 32 / 8;       // >= 2 blocks per wave
    const int by_fill = (512 + pairs - 1) / pairs;         // aim at ~512 workgroups
    p.splits = at_most(most, by_fill);
  } else if (T == 15 && 8 * pairs <= 3 * cus) {
    int most = 4;
    if (8 * pairs <= cus) most = at_least(6, at_most(by_len, full_splits(g, B, pairs)));
    else if (B <= 2 && 4 * pairs <= cus && max_prefix >= 4096) most = at_least(6, cus / pairs);
    else if (3 * pairs <= cus && max_prefix >= 2560) most = cus / pairs;
    p.splits = at_most(nb / 6, most);
  } else if (2 * pairs <= cus) {
    if (T == 15)
      p.splits = at_most(by_len, cus / pairs);
    else if (p.halves)
      p.splits = halves_splits(B, pairs, max_prefix, g.group > 1);
    else
      p.splits = at_most(1 + (int)sqrtf((float)nb / 4.0f), g.quant ? cus / pairs : full_splits(g, B, pairs));
  }
#ifdef MDZ_DEV_KNOBS
  static const char* env_s = getenv("MDZ_ATTN_SPLITS");  // development builds only
  if (env_s && atoi(env_s) > 0) p.splits = atoi(env_s);
  static const char* env_h = getenv("MDZ_ATTN_HALVES");  // 1 = 32 queries per workgroup, 0 = 64
  if (env_h && T == 64) p.halves = atoi(env_h) != 0;
#endif
  p.splits = p.splits < 1 ? 1 : p.splits > 32 ? 32 : p.splits;
  // Long sequences first, where the launch gains by it: finding its place costs a workgroup 1 - 2 us, and where all workgroups run at
  // once the hardware's order pairs them better.  us per layer, lengths S / 4 .. S, in order / not, 64 nodes unless said otherwise:
  //   one split, more workgroups than fit (32 heads): 32 sequences at S = 1000 135 / 124, 2000 194 / 188, 3000 255 / 256, 4000 315 / 328;
  //     16 at 1000 64 / 62, 3000 131 / 134, 4000 168 / 174; 8-bit rows: 32 at 1000 119 / 117, 2000 157 / 162, 16 at 1000 57 / 59, 2000 75 / 84;
  //     15 nodes, 32 at 250 35 / 33, 1000 81 / 85, 4000 257 / 268;
  //   one split, all at once: 6 at 1000 31 / 27, 3000 64 / 58 (15 nodes gain: 12 at 1000 32 / 33, 3000 87 / 92);
  //   several splits: 3 at 1000 24.5 / 23.6, 2000 26.9 / 28.9, 3000 34.5 / 38.0, 8-bit rows at 6000 38 / 44.
  const int halves_of_tree = T == 64 && p.halves ? 2 : 1;
  const int64_t wgs = (int64_t)p.splits * pairs * halves_of_tree;
  p.ordered = B > 1 && (p.splits > 1 ? wgs > cus && max_prefix >= 1536
                                     : wgs > halves_of_tree * cus && max_prefix >= (T == 64 && !g.quant ? 2560 : 1024));
  return p;
}

AttentionPlan attn_mfma_plan(int tree, const KvGeom& g, int B, int max_prefix, bool fused) {
  const AttnPlan p = attn_plan(host_tree(tree)->T, g, B, max_prefix, fused);
  return AttentionPlan{ATTN_TREE, host_tree(tree)->T == 64 && !p.halves ? 64 : 32, p.splits, p.ordered};
}

// Scratch of the splits' partial outputs.  A workspace is sized before the cache's row type is known and may serve shorter prefixes than it was
// sized for: the most splits of any plan for up to max_prefix keys.  Each rule's count grows with the prefix, but from 32 to 64 queries and, for
// 15 nodes, at 2560 keys.
int64_t attn_mfma_scratch_bytes(int B, const KvGeom& g, int T, int max_prefix) {
  const int pairs = B * q_heads(g);
  int most = attn_plan(T, g, B, max_prefix, false).splits;
  for (int quant = 0; quant < 2; ++quant) {
    KvGeom gq = g;
    gq.quant = quant;
    const int s = attn_plan(T, gq, B, max_prefix, true).splits;
    if (s > most) most = s;
  }
  if (T == 64 && 2 * pairs <= num_cus()) {
    const int s = halves_splits(B, pairs, max_prefix, g.group > 1);
    if (s > most) most = s;
  }
  if (T == 15 && max_prefix >= 2560) {
    const int s = attn_plan(T, g, B, 2559, true).splits;
    if (s > most) most = s;
  }
#ifdef MDZ_DEV_KNOBS
  most = 32;
#endif
  return most == 1 ? 0 : (int64_t)pairs * most * (T * kHD + 2 * T) * 4;
}

template <typename E, bool Q8, int NU, int TQ, bool ONCE>
static int launch_attention_mfma_t(int tree, const void* q, const Partials* qkv, const float* cs, const KvGeom& g, void* kc,
                                   void* vc, int layer, const int32_t* seq_len, int B, int max_prefix, const AttnPlan& p, void* att_out,
                                   void* scratch, int64_t scratch_bytes, hipStream_t st) {
  // the merge buffer [4][128][32 NU + 2] + [4][2][32 NU] floats overlays the staged Q tile and tree rows
  constexpr int lds_bytes = 4 * kHD * (32 * NU + 2) * 4 + 4 * 2 * 32 * NU * 4;
  static_assert(lds_bytes >= (32 * NU + 2 * TQ) * kQRow && lds_bytes * (3 - NU) <= 160 * 1024, "LDS budget of the tree kernel");
  MDZ_SET_LDS_ONCE((attn_tree_mfma_kernel<E, Q8, NU, TQ, ONCE>), lds_bytes);
  const int nq = q_heads(g), splits = p.splits;
  MDZ_REQUIRE(scratch_bytes >= attn_mfma_scratch_bytes(B, g, TQ, max_prefix), MDZ_EWORKSPACE, "attention: scratch too small");
  float* part_o = (float*)scratch;
  float* part_ml = part_o + (int64_t)B * nq * splits * TQ * kHD;
  dim3 grid(splits, nq, B * (TQ > 32 * NU ? 2 : 1));  // two workgroups share a sequence: blockIdx.z = 2 * sequence + half
  const Partials none = single_slot(nullptr, 0, 0);
  launch_timed(PROF_ATTN, attn_tree_mfma_kernel<E, Q8, NU, TQ, ONCE>, grid, 256, lds_bytes, st, tree, (const E*)q, qkv ? *qkv : none, cs, g,
               (E*)kc, (E*)vc, layer, seq_len, max_prefix, (E*)att_out, part_o, part_ml, p.ordered);
  MDZ_LAUNCH_CHECK();
  if (splits > 1) {
    launch_timed(PROF_ATTN, attn_combine_kernel<E, TQ>, dim3(nq, B, (TQ + 15) / 16), 256, 0, st, nq, splits, part_o, part_ml, (E*)att_out);
    MDZ_LAUNCH_CHECK();
  }
  return MDZ_OK;
}

int launch_attention_mfma(int dtype, int tree, const void* q, const Partials* qkv, const float* cs, const KvGeom& g,
                          void* kc, void* vc, int layer, const int32_t* seq_len, int B, int max_prefix, void* att_out,
                          void* scratch, int64_t scratch_bytes, hipStream_t st) {
  if (B == 0) return MDZ_OK;
  const int T = host_tree(tree)->T;
  const AttnPlan p = attn_plan(T, g, B, max_prefix, qkv != nullptr);
  const bool once = g.group == 1;  // (and not in halves; 8-bit rows run alike: 16K keys 801 / 802 us per step of 4 layers)
#define MDZ_ATTN_CASE(Q8, NU, TQ, ONCE)                                                                                     \
  MDZ_WITH_ELEM16(dtype, return (launch_attention_mfma_t<E, Q8, NU, TQ, ONCE>(tree, q, qkv, cs, g, kc, vc, layer, seq_len, B, \
                                                                              max_prefix, p, att_out, scratch, scratch_bytes, st)))
  if (T == 15) {
    if (once) MDZ_ATTN_CASE(false, 1, 15, true);
    MDZ_ATTN_CASE(false, 1, 15, false);
  }
  if (g.quant) {
    if (p.halves) MDZ_ATTN_CASE(true, 1, 64, false);
    MDZ_ATTN_CASE(true, 2, 64, false);
  }
  if (p.halves) MDZ_ATTN_CASE(false, 1, 64, false);
  if (once) MDZ_ATTN_CASE(false, 2, 64, true);
  MDZ_ATTN_CASE(false, 2, 64, false);
#undef MDZ_ATTN_CASE
}

}  // namespace mdz
