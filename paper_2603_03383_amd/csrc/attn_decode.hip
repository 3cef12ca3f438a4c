// Single-query attention over the tiled 16-bit (bf16 or fp16) KV cache: the degenerate tree of one node, i.e. one ordinary
// autoregressive decode step (Section 4.1: the Time_AR that the paper's Overhead and Speedup are measured
// against).  The node sees the prefix and itself, so the mask is "slot <= S".
//
// One workgroup = 4 waves handles one (sequence, KEY/VALUE head, key-split): the query heads of a group are the columns of one
// 32-column operand, so grouped heads read K and V once (one query head per workgroup read them `group` times: 92 us per
// layer for 24 sequences of 90 .. 3000 keys with 8 key/value and 32 query heads, 37 us now).  A wave walks 32-key blocks of
// the tiled cache (common.h) with contiguous 16-byte-per-lane loads that are MFMA A operands as they are; scores are
// computed transposed (keys x queries), so the probabilities of 16 keys of one query sit in a lane and feed the second
// MFMA from registers, as in the tree kernel, but as the 16-bit terms of their fp32 values (WeightTerms).  Columns beyond the
// group's heads are zero and never stored: the matrix cores idle otherwise, the kernel is bound by the K / V stream and, at short
// prefixes, by its fixed chain (many sequences of ungrouped heads: attn_decode_one_kernel below).
// The kernel starts from the QKV GEMM's partial sums: every workgroup reduces and rotates the queries of its group; the
// split that owns the block of slot S also produces the node's K and V rows, writes them to the cache and puts them into
// the block from LDS, so that no load waits for a store (a launch of its own took 4.9 us per layer).  Waves merge
// through LDS, key-splits through a second small kernel, both in a fixed order.
// Q8 = true: 8-bit rows (common.h): a block is 4 K units + 4 V units + 2 x 32 scales; K codes convert exactly to E in registers and
// the K scales multiply the scores in fp32.  The V scales multiply the probabilities in fp32 too; a scale is |row| / 448, so
// that product is split into bf16 terms, which have fp32's range, and the V codes convert exactly to bf16, in fp16 models too.
#include <type_traits>

#include "kernels.h"

namespace mdz {

typedef u32x4_t u32x4;
typedef f32x16_t f32x16;

namespace {
constexpr int kHD = 128;
constexpr int kQRow = kHD * 2 + 16;  // bytes per staged query row
constexpr int kORow = kHD + 4;       // floats per merged output row

// Two adjacent columns and their rotary partners (64 columns on) of one row of the QKV partial sums.  load() requests the
// first kEarly slots, sum() adds the slots in order and fetches what lies beyond kEarly, behind the first K / V block.  (A 4096-wide
// model's product has two slots; narrow ones have more, e.g. eight at 1024, and pay that second round trip.)
struct PairSums {
  static constexpr int kEarly = 4;
  float2 a[kEarly], p[kEarly];
  const float* src;
  int n;
  __device__ inline void load(const Partials& part, int64_t row, int col) {
    n = part.count(col);
    src = part.p + row * part.ld + col;
#pragma unroll
    for (int s = 0; s < kEarly; ++s)
      if (s < n) {
        a[s] = *reinterpret_cast<const float2*>(src + (int64_t)s * part.stride);
        p[s] = *reinterpret_cast<const float2*>(src + (int64_t)s * part.stride + 64);
      }
  }
  __device__ inline void sum(const Partials& part, float2& ra, float2& rp) const {
    ra = rp = float2{0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kEarly; ++s)
      if (s < n) ra.x += a[s].x, ra.y += a[s].y, rp.x += p[s].x, rp.y += p[s].y;
    for (int s = kEarly; s < n; ++s) {
      const float2 va = *reinterpret_cast<const float2*>(src + (int64_t)s * part.stride);
      const float2 vp = *reinterpret_cast<const float2*>(src + (int64_t)s * part.stride + 64);
      ra.x += va.x, ra.y += va.y, rp.x += vp.x, rp.y += vp.y;
    }
  }
};
__device__ inline void rotate(const float4& t, float2& a, float2& p) {  // t: cos, sin of the two pairs
  const float2 ra = {a.x * t.x - p.x * t.y, a.y * t.z - p.y * t.w};
  p = float2{p.x * t.x + a.x * t.y, p.y * t.z + a.y * t.w};
  a = ra;
}

// Threads 192 .. 255 of the workgroup: the node's K row (192 .. 223) and V row from their QKV sums, two rotary pairs per thread
// (features f, f + 1 and f + 64, f + 65), to the cache and to kv_lds (K row, then kQRow bytes on the V row: 128 elements; 8-bit
// rows: 128 codes, scale).
template <typename E, bool Q8>
__device__ inline void write_own_row(const Partials& qkv, const PairSums& kvs, const float4& rot, uint8_t* kv_lds, const KvGeom& g,
                                     E* kc, E* vc, int layer, int b, int hk, int S) {
  const int tid = threadIdx.x, f = (tid & 31) * 2;
  const bool is_k = tid < 224;
  uint8_t* stage = kv_lds + (is_k ? 0 : kQRow);
  float2 a, p;
  kvs.sum(qkv, a, p);
  if (is_k) rotate(rot, a, p);
  if constexpr (Q8) {
    float am = fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(p.x), fabsf(p.y)));
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) am = fmaxf(am, __shfl_xor(am, o, 64));  // over the 32 threads of the row
    const float sc = kv8_scale_of(am);
    const uint32_t w = kv8_pack4(a.x, a.y, p.x, p.y, sc);
    *reinterpret_cast<uint16_t*>(stage + f) = (uint16_t)w;
    *reinterpret_cast<uint16_t*>(stage + 64 + f) = (uint16_t)(w >> 16);
    uint8_t* dst = reinterpret_cast<uint8_t*>(is_k ? kc : vc) + kv8_head_base(g, layer, b, hk);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = f + (e & 1) + (e >> 1) * 64;
      dst[is_k ? kv8_k_code(S, i) : kv8_v_code(S, i)] = (uint8_t)(w >> (8 * e));
    }
    if ((tid & 31) == 0) {
      *reinterpret_cast<float*>(dst + kv8_scale(S)) = sc;
      *reinterpret_cast<float*>(stage + 128) = sc;
    }
  } else {
    const uint32_t lo = Elem16<E>::pack2(a.x, a.y), hi = Elem16<E>::pack2(p.x, p.y);
    *reinterpret_cast<uint32_t*>(stage + 2 * f) = lo;
    *reinterpret_cast<uint32_t*>(stage + 128 + 2 * f) = hi;
    if (is_k) {  // adjacent features of one key are adjacent in the tiled K layout
      *reinterpret_cast<uint32_t*>(kc + k_index(g, layer, b, hk, S, f)) = lo;
      *reinterpret_cast<uint32_t*>(kc + k_index(g, layer, b, hk, S, f + 64)) = hi;
    } else {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        vc[v_index(g, layer, b, hk, S, f + e)] = E{(uint16_t)(lo >> (16 * e))};
        vc[v_index(g, layer, b, hk, S, f + 64 + e)] = E{(uint16_t)(hi >> (16 * e))};
      }
    }
  }
}

// Puts the node's own row, staged in LDS, into the units of the block that holds slot S (its cache copy may not have arrived
// yet).  Lane (key, gh) of a K unit, lane (feature % 32 = key, gh) of a V unit; own = S % 32.
template <bool Q8, int N>
__device__ inline void put_own_row(const uint8_t* kv_lds, int key, int gh, int own, u32x4 (&kd)[N], u32x4 (&vd)[N]) {
  const bool mine = ((own >> 2) & 1) == gh;  // V units: the half-wave that holds key `own`
  if constexpr (Q8) {
    if (key == own) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint2 lo = *reinterpret_cast<const uint2*>(kv_lds + 32 * j + 8 * gh);
        const uint2 hi = *reinterpret_cast<const uint2*>(kv_lds + 32 * j + 16 + 8 * gh);
        kd[j] = u32x4{lo.x, lo.y, hi.x, hi.y};
      }
    }
    const int byte = 8 * (own >> 4) + 4 * ((own >> 3) & 1) + (own & 3);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t code = kv_lds[kQRow + 32 * t + key];
#pragma unroll
      for (int w = 0; w < 4; ++w)
        if (mine && w == byte >> 2) vd[t][w] = (vd[t][w] & ~(0xFFu << (8 * (byte & 3)))) | code << (8 * (byte & 3));
    }
  } else {
    if (key == own) {
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) kd[ks] = *reinterpret_cast<const u32x4*>(kv_lds + 32 * ks + 16 * gh);
    }
    const int e = 4 * ((own >> 3) & 1) + (own & 3), sh = 16 * (e & 1);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t v = *reinterpret_cast<const uint16_t*>(kv_lds + kQRow + 2 * (32 * t + key));
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int w = 0; w < 4; ++w)
          if (mine && s2 == own >> 4 && w == e >> 1) vd[2 * t + s2][w] = (vd[2 * t + s2][w] & ~(0xFFFFu << sh)) | v << sh;
    }
  }
}

// 8 elements, or 8 E4M3 codes (words 2 * half, 2 * half + 1 of v), as floats
template <typename E>
__device__ inline void unpack8(u32x4 v, float (&f)[8]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) f[2 * i] = Elem16<E>::lo(v[i]), f[2 * i + 1] = Elem16<E>::hi(v[i]);
  // Keeps the conversions as instructions of their own: for fp16 the compiler otherwise folds them into mixed-precision FMAs
  // (v_fma_mix_f32), which run at a third of the speed here.
#pragma unroll
  for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(f[i]));
}
__device__ inline void unpack8_fp8(u32x4 v, int half, float (&f)[8]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t w = v[2 * half + i];
    const auto a = __builtin_amdgcn_cvt_pk_f32_fp8(w, false), c = __builtin_amdgcn_cvt_pk_f32_fp8(w, true);
    f[4 * i] = a[0], f[4 * i + 1] = a[1], f[4 * i + 2] = c[0], f[4 * i + 3] = c[1];
  }
}
}  // namespace

// qkv.p == NULL: q [B][d] holds the rotated queries and the cache already holds the node's row (separate RoPE kernel).
template <typename E, bool Q8, bool ONCE>
__global__ void __launch_bounds__(256, 2)
    attn_decode_kernel(const E* __restrict__ q, const Partials qkv, const float* __restrict__ cs, KvGeom g, E* __restrict__ kc,
                       E* __restrict__ vc, int layer, const int32_t* __restrict__ seq_len, int max_prefix,
                       E* __restrict__ att_out, float* __restrict__ part_o, float* __restrict__ part_ml, bool ordered) {
  extern __shared__ __attribute__((aligned(16))) uint8_t lds_raw[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int qi = lane & 31, gh = lane >> 5;
  const int split = blockIdx.x, n_splits = gridDim.x;
  const int b = ordered ? sequence_in_order(seq_len, gridDim.z, blockIdx.z) : blockIdx.z;
  const int chunks = (g.group + 31) >> 5;  // groups of more than 32 query heads take several workgroups
  const int hk = blockIdx.y / chunks, h0 = hk * g.group + (blockIdx.y % chunks) * 32;
  const int nq = min(32, g.group - (blockIdx.y % chunks) * 32);  // query heads of this workgroup: h0 .. h0 + nq - 1
  const int d = q_heads(g) * kHD, dkv = g.n_heads * kHD;
  const int S = min(max(seq_len[b], 0), max_prefix);
  const int nb = (S + 1 + 31) >> 5;
  const int blk_begin = (int)((int64_t)split * nb / n_splits), blk_end = (int)((int64_t)(split + 1) * nb / n_splits);

  // 16-bit rows: block blk, unit i at kp[blk*512 + i*64].  8-bit rows: at kp[blk*264 + i*64], the four scales of keys
  // 8j + 4gh .. +3 at ks_p[blk*264 + 2j]
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
  // K and V double buffered one block ahead; every load is unconditional (past the wave's last block it repeats it)
  u32x4 kb[2][8], vb[2][8];
  auto unit = [](const u32x4* p) { return ONCE ? __builtin_nontemporal_load(p) : *p; };
  auto load_kv = [&](int blk, u32x4 (&kd)[8], u32x4 (&vd)[8]) {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      kd[i] = (Q8 && i >= 4) ? ks_p[(int64_t)blk * kBlkPieces + 2 * (i - 4)] : unit(kp + (int64_t)blk * kBlkPieces + i * 64);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      vd[i] = (Q8 && i >= 4) ? vs_p[(int64_t)blk * kBlkPieces + 2 * (i - 4)] : unit(vp + (int64_t)blk * kBlkPieces + i * 64);
  };
  // Requested first (loads return in order): the partial sums of two rotary pairs of one query head per thread, and, in the
  // split that owns the block of slot S, the node's K row (threads 192 .. 223) and V row (224 .. 255).
  const bool fused = qkv.p != nullptr, owner = blk_begin < blk_end && blk_end == nb;
  const float* csr = cs + (int64_t)b * kHD;  // [64 pairs][cos, sin]
  const int f = (tid & 31) * 2;              // first of the thread's two features; partners 64 further
  PairSums qs, kvs;
  float4 rot = {};
  if (fused) {
    rot = *reinterpret_cast<const float4*>(csr + 2 * f);
    if ((tid >> 5) < nq) qs.load(qkv, b, (h0 + (tid >> 5)) * kHD + f);
    if (owner && tid >= 192) kvs.load(qkv, b, d + (tid < 224 ? 0 : dkv) + hk * kHD + f);
  }
  const int n_mine = blk_begin + wave < blk_end ? (blk_end - blk_begin - wave + 3) >> 2 : 0;
  const int first = blk_begin + wave, last = first + 4 * (n_mine - 1);
  // The first block waits for nothing below: the node's own row, if it falls into it, is put in from LDS.
  __builtin_amdgcn_sched_barrier(0);
  if (n_mine > 0) load_kv(first, kb[0], vb[0]);
  __builtin_amdgcn_sched_barrier(0);

  // queries -> LDS, rows beyond nq zero
  uint8_t* q_lds = lds_raw;
  uint8_t* kv_lds = lds_raw + 32 * kQRow;  // the node's K row, then its V row: 128 elements (8-bit rows: 128 codes, scale)
  if (!fused) {
    for (int i = tid; i < 32 * 16; i += 256) {
      const int row = i >> 4, c = i & 15;
      u32x4 v = {0, 0, 0, 0};
      if (row < nq) v = *reinterpret_cast<const u32x4*>(q + (int64_t)b * d + (h0 + row) * kHD + c * 8);
      *reinterpret_cast<u32x4*>(q_lds + row * kQRow + c * 16) = v;
    }
  } else {
    for (int row = tid >> 5; row < 32; row += 8) {
      uint32_t lo = 0, hi = 0;
      if (row < nq) {
        if (row >= 8) qs.load(qkv, b, (h0 + row) * kHD + f);
        float2 a, p;
        qs.sum(qkv, a, p);
        rotate(rot, a, p);
        lo = Elem16<E>::pack2(a.x, a.y), hi = Elem16<E>::pack2(p.x, p.y);
      }
      *reinterpret_cast<uint32_t*>(q_lds + row * kQRow + 2 * f) = lo;
      *reinterpret_cast<uint32_t*>(q_lds + row * kQRow + 128 + 2 * f) = hi;
    }
    if (owner && tid >= 192) write_own_row<E, Q8>(qkv, kvs, rot, kv_lds, g, kc, vc, layer, b, hk, S);
  }
  __syncthreads();

  const int own_blk = fused ? S >> 5 : -1, own = S & 31;
  auto put_own = [&](u32x4 (&kd)[8], u32x4 (&vd)[8]) {
    put_own_row<Q8>(kv_lds, qi, gh, own, kd, vd);
    if constexpr (Q8) {  // its scales: the half-wave that holds key `own`
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (((own >> 2) & 1) == gh && t == own >> 3 && e == (own & 3)) {
            kd[4 + t][e] = *reinterpret_cast<const uint32_t*>(kv_lds + 128);
            vd[4 + t][e] = *reinterpret_cast<const uint32_t*>(kv_lds + kQRow + 128);
          }
    }
  };

  const uint8_t* qfrag = q_lds + qi * kQRow + gh * 16;  // B operand of scores^T: query qi, features 16 ks + 8 gh .. +7
  const float scale_log2 = 1.4426950408889634f / sqrtf((float)kHD);
  float m_run = -INFINITY, l_run = 0.f;
  f32x16 o[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.f;

  using VE = std::conditional_t<Q8, bf16_t, E>;  // operand type of the product with V
  auto process = [&](int blk, const u32x4 (&kd)[8], const u32x4 (&vd)[8]) {
    // Compiler barrier: keeps the (loop-invariant) query operands in LDS instead of in 32 registers this kernel lacks
    asm volatile("" ::: "memory");
    f32x16 sc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const u32x4 ka = Q8 ? fp8x8_to_elem<E>(kd[ks >> 1], ks & 1) : kd[ks];
      sc = Elem16<E>::mfma(ka, *reinterpret_cast<const u32x4*>(qfrag + ks * 32), sc);
    }
    // register r is key 8*(r/4) + 4*gh + r%4 of the block; its scale is component r%4 of scale piece r/4
    float bmax = -INFINITY;
    const int left = S + 1 - blk * 32 - 4 * gh;  // keys of this half-wave's numbering that are visible
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float s = sc[r] * (Q8 ? __uint_as_float(kd[4 + (r >> 2)][r & 3]) * scale_log2 : scale_log2);
      s = 8 * (r >> 2) + (r & 3) < left ? s : -INFINITY;
      sc[r] = s;
      bmax = fmaxf(bmax, s);
    }
    bmax = fmaxf(bmax, __shfl_xor(bmax, 32, 64));  // finite: a block in range holds at least one visible slot
    const float m_new = fmaxf(m_run, bmax);
    const float alpha = fast_exp2(m_run - m_new);
    float sum = 0.f, p[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) p[r] = fast_exp2(sc[r] - m_new) * WeightTerms<VE>::kScale;
#pragma unroll
    for (int r = 0; r < 16; r += 2) sum += p[r] + p[r + 1];
    if constexpr (Q8) {  // a slot that no row was ever written to may hold any finite scale; its probability is zero
#pragma unroll
      for (int r = 0; r < 16; ++r) p[r] *= __uint_as_float(vd[4 + (r >> 2)][r & 3]);
    }
    l_run = l_run * alpha + sum;
    if (__any(m_new != m_run)) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
    }
    m_run = m_new;
#pragma unroll
    for (int i = 0; i < WeightTerms<VE>::kTerms; ++i) {
      u32x4 pf[2];
      next_weight_term<VE>(p, pf);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          const u32x4 va = Q8 ? fp8x8_to_elem<VE>(vd[t], s2) : vd[t * 2 + s2];
          o[t] = Elem16<VE>::mfma(va, pf[s2], o[t]);
        }
    }
  };
  if (n_mine > 0) {
    for (int it = 0; it < n_mine; it += 2) {
      const int blk = first + 4 * it;
      load_kv(min(blk + 4, last), kb[1], vb[1]);
      __builtin_amdgcn_sched_barrier(0);
      if (blk == own_blk) put_own(kb[0], vb[0]);
      process(blk, kb[0], vb[0]);
      __builtin_amdgcn_sched_barrier(0);
      load_kv(min(blk + 8, last), kb[0], vb[0]);
      __builtin_amdgcn_sched_barrier(0);
      if (it + 1 < n_mine) {
        if (blk + 4 == own_blk) put_own(kb[1], vb[1]);
        process(blk + 4, kb[1], vb[1]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- merge the four waves (fixed order), then store or hand the partial result to the combine kernel
  __syncthreads();  // every wave has its query operands; the merge buffer overlays them
  float* o_lds = reinterpret_cast<float*>(lds_raw);  // [4][nq][kORow]
  float* m_lds = o_lds + 4 * nq * kORow;             // [4][nq]
  float* l_lds = m_lds + 4 * nq;
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (qi < nq) {
    if (gh == 0) m_lds[wave * nq + qi] = m_run, l_lds[wave * nq + qi] = l_tot;
    float* dst = o_lds + (wave * nq + qi) * kORow + 4 * gh;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        *reinterpret_cast<float4*>(dst + 32 * t + 8 * c) = float4{o[t][4 * c], o[t][4 * c + 1], o[t][4 * c + 2], o[t][4 * c + 3]};
  }
  __syncthreads();
  for (int i = tid; i < nq * 32; i += 256) {  // thread: 4 features of one query head
    const int qq = i >> 5, f = (i & 31) * 4;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < 4; ++w) M = fmaxf(M, m_lds[w * nq + qq]);
    const float M_safe = M == -INFINITY ? 0.f : M;
    float L = 0.f;
    float4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float wt = fast_exp2(m_lds[w * nq + qq] - M_safe);
      const float4 v = *reinterpret_cast<const float4*>(o_lds + (w * nq + qq) * kORow + f);
      L += wt * l_lds[w * nq + qq];
      a.x += wt * v.x, a.y += wt * v.y, a.z += wt * v.z, a.w += wt * v.w;
    }
    if (n_splits == 1) {
      const float inv = 1.0f / L;
      *reinterpret_cast<uint2*>(att_out + (int64_t)b * d + (h0 + qq) * kHD + f) =
          uint2{Elem16<E>::pack2(a.x * inv, a.y * inv), Elem16<E>::pack2(a.z * inv, a.w * inv)};
    } else {
      const int64_t pidx = (int64_t)(b * q_heads(g) + h0 + qq) * n_splits + split;
      *reinterpret_cast<float4*>(part_o + pidx * kHD + f) = a;
      if (f == 0) part_ml[pidx * 2] = M, part_ml[pidx * 2 + 1] = L;
    }
  }
}

// The same for ungrouped heads where more workgroups are asked for than the kernel above keeps resident (two per CU): one query
// leaves 31 of the MFMA's 32 columns and most of that kernel's registers idle, and with many short sequences its time is the chain of
// each workgroup, of which a CU then works on two.  Here the products are fp32 FMAs: lane (key, gh) of a K unit has half the
// features of key `key`, lane (feature % 32, gh) of a V unit 16 of the 32 keys; four workgroups share a CU, and the next block's K
// (V) is requested as soon as this block's registers are free.
template <typename E, bool Q8>
__global__ void __launch_bounds__(256, 4)
    attn_decode_one_kernel(const E* __restrict__ q, const Partials qkv, const float* __restrict__ cs, KvGeom g, E* __restrict__ kc,
                           E* __restrict__ vc, int layer, const int32_t* __restrict__ seq_len, int max_prefix,
                           E* __restrict__ att_out, float* __restrict__ part_o, float* __restrict__ part_ml, bool ordered) {
  __shared__ __attribute__((aligned(16))) float q_lds[kHD];
  __shared__ __attribute__((aligned(16))) uint8_t kv_lds[2 * kQRow];
  __shared__ __attribute__((aligned(16))) float p_lds[4][32];
  __shared__ float o_lds[4][kHD], m_lds[4], l_lds[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int key = lane & 31, gh = lane >> 5;
  const int split = blockIdx.x, n_splits = gridDim.x, h = blockIdx.y;
  const int b = ordered ? sequence_in_order(seq_len, gridDim.z, blockIdx.z) : blockIdx.z;
  const int d = g.n_heads * kHD;
  const int S = min(max(seq_len[b], 0), max_prefix);
  const int nb = (S + 1 + 31) >> 5;
  const int blk_begin = (int)((int64_t)split * nb / n_splits), blk_end = (int)((int64_t)(split + 1) * nb / n_splits);

  constexpr int kUnits = Q8 ? 4 : 8, kBlkPieces = Q8 ? kKv8BlockBytes / 16 : 512;
  const uint8_t* kbase = reinterpret_cast<const uint8_t*>(kc) + (Q8 ? kv8_head_base(g, layer, b, h) : kv_head_base(g, layer, b, h) * 2);
  const uint8_t* vbase = reinterpret_cast<const uint8_t*>(vc) + (Q8 ? kv8_head_base(g, layer, b, h) : kv_head_base(g, layer, b, h) * 2);
  const u32x4* kp = reinterpret_cast<const u32x4*>(kbase) + lane;
  const u32x4* vp = reinterpret_cast<const u32x4*>(vbase) + lane;
  // Read once per pass, by no other workgroup, so non-temporally (us per step of 4 layers, plain / non-temporal: 20 sequences of 200 .. 2000
  // keys 818 / 791, 64 of 40 .. 400 798 / 783, 90 of 300 .. 3000 at 16 heads 1223 / 1152).
  u32x4 kd[kUnits], vd[kUnits];
  float k_scale = 1.f, v_scale = 1.f;  // 8-bit rows: of key `key`
  auto load_k = [&](int blk) {
#pragma unroll
    for (int i = 0; i < kUnits; ++i) kd[i] = __builtin_nontemporal_load(kp + (int64_t)blk * kBlkPieces + i * 64);
    if constexpr (Q8) k_scale = *reinterpret_cast<const float*>(kbase + (int64_t)blk * kKv8BlockBytes + 4096 + key * 4);
  };
  auto load_v = [&](int blk) {
#pragma unroll
    for (int i = 0; i < kUnits; ++i) vd[i] = __builtin_nontemporal_load(vp + (int64_t)blk * kBlkPieces + i * 64);
    if constexpr (Q8) v_scale = *reinterpret_cast<const float*>(vbase + (int64_t)blk * kKv8BlockBytes + 4096 + key * 4);
  };

  // (order of requests and hand-over of the node's own row: as above)
  const bool fused = qkv.p != nullptr, owner = blk_begin < blk_end && blk_end == nb;
  const int f = (tid & 31) * 2;
  PairSums sums;
  float4 rot = {};
  if (fused && (tid < 32 || (owner && tid >= 192))) {
    rot = *reinterpret_cast<const float4*>(cs + (int64_t)b * kHD + 2 * f);
    sums.load(qkv, b, (tid < 32 ? 0 : tid < 224 ? d : 2 * d) + h * kHD + f);
  }
  const int n_mine = blk_begin + wave < blk_end ? (blk_end - blk_begin - wave + 3) >> 2 : 0;
  const int first = blk_begin + wave, last = first + 4 * (n_mine - 1);
  __builtin_amdgcn_sched_barrier(0);
  if (n_mine > 0) load_k(first), load_v(first);
  __builtin_amdgcn_sched_barrier(0);
  if (!fused) {
    if (tid < kHD) q_lds[tid] = to_float(q[(int64_t)b * d + h * kHD + tid]);
  } else if (tid < 32) {  // the query as the storage type holds it
    float2 a, p;
    sums.sum(qkv, a, p);
    rotate(rot, a, p);
    const uint32_t lo = Elem16<E>::pack2(a.x, a.y), hi = Elem16<E>::pack2(p.x, p.y);
    q_lds[f] = Elem16<E>::lo(lo), q_lds[f + 1] = Elem16<E>::hi(lo);
    q_lds[f + 64] = Elem16<E>::lo(hi), q_lds[f + 65] = Elem16<E>::hi(hi);
  } else if (owner && tid >= 192) {
    write_own_row<E, Q8>(qkv, sums, rot, kv_lds, g, kc, vc, layer, b, h, S);
  }
  __syncthreads();

  const float scale_log2 = 1.4426950408889634f / sqrtf((float)kHD);
  float m_run = -INFINITY, l_run = 0.f;  // l_run: of this lane's keys
  float o[4] = {0.f, 0.f, 0.f, 0.f};     // feature 32 t + key, over the keys this half-wave holds
  auto process = [&](int blk, auto is_last) {  // is_last: the wave's last block, the only one that can hold slot S and slots beyond it
    if constexpr (decltype(is_last)::value) {
      if (fused && blk == S >> 5) {
        put_own_row<Q8>(kv_lds, key, gh, S & 31, kd, vd);
        if constexpr (Q8) {
          if (key == (S & 31)) {
            k_scale = *reinterpret_cast<const float*>(kv_lds + 128);
            v_scale = *reinterpret_cast<const float*>(kv_lds + kQRow + 128);
          }
        }
      }
    }
    asm volatile("" ::: "memory");  // keeps the query in LDS, out of 64 registers
    float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {  // features 16 ks + 8 gh .. +7
      float k8[8];
      if constexpr (Q8) unpack8_fp8(kd[ks >> 1], ks & 1, k8);
      else unpack8<E>(kd[ks], k8);
      const float4 qa = *reinterpret_cast<const float4*>(q_lds + 16 * ks + 8 * gh);
      const float4 qb = *reinterpret_cast<const float4*>(q_lds + 16 * ks + 8 * gh + 4);
      part[0] += qa.x * k8[0], part[1] += qa.y * k8[1], part[2] += qa.z * k8[2], part[3] += qa.w * k8[3];
      part[0] += qb.x * k8[4], part[1] += qb.y * k8[5], part[2] += qb.z * k8[6], part[3] += qb.w * k8[7];
    }
    float s = (part[0] + part[1]) + (part[2] + part[3]);
    s = (s + __shfl_xor(s, 32, 64)) * (Q8 ? k_scale * scale_log2 : scale_log2);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!decltype(is_last)::value) load_k(blk + 4);
    else s = blk * 32 + key <= S ? s : -INFINITY;
    __builtin_amdgcn_sched_barrier(0);
    float bmax = s;
#pragma unroll
    for (int x = 16; x > 0; x >>= 1) bmax = fmaxf(bmax, __shfl_xor(bmax, x, 64));
    const float m_new = fmaxf(m_run, bmax);  // finite: a block in range holds at least one visible slot
    const float alpha = fast_exp2(m_run - m_new), p = fast_exp2(s - m_new);
    l_run = l_run * alpha + p;
    m_run = m_new;
    p_lds[wave][key] = Q8 ? p * v_scale : p;  // (a slot that no row was ever written to may hold any finite scale; its p is zero)
    __builtin_amdgcn_wave_barrier();
    float4 pk[4];  // keys 8 c + 4 gh .. +3
#pragma unroll
    for (int c = 0; c < 4; ++c) pk[c] = *reinterpret_cast<const float4*>(&p_lds[wave][8 * c + 4 * gh]);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float a = o[t] * alpha;
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        float v8[8];
        if constexpr (Q8) unpack8_fp8(vd[t], s2, v8);
        else unpack8<E>(vd[2 * t + s2], v8);
        const float4 pa = pk[2 * s2], pb = pk[2 * s2 + 1];
        a += pa.x * v8[0], a += pa.y * v8[1], a += pa.z * v8[2], a += pa.w * v8[3];
        a += pb.x * v8[4], a += pb.y * v8[5], a += pb.z * v8[6], a += pb.w * v8[7];
      }
      o[t] = a;
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!decltype(is_last)::value) load_v(blk + 4);
    __builtin_amdgcn_sched_barrier(0);
  };
  if (n_mine > 0) {
    for (int blk = first; blk < last; blk += 4) process(blk, std::false_type{});
    process(last, std::true_type{});
  }

  // ---- merge the four waves (fixed order), then store or hand the partial result to the combine kernel
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    o[t] += __shfl_xor(o[t], 32, 64);
    if (gh == 0) o_lds[wave][32 * t + key] = o[t];
  }
#pragma unroll
  for (int x = 16; x > 0; x >>= 1) l_run += __shfl_xor(l_run, x, 64);
  if (lane == 0) m_lds[wave] = m_run, l_lds[wave] = l_run;
  __syncthreads();
  if (tid >= kHD) return;
  float M = -INFINITY, L = 0.f, a = 0.f;
#pragma unroll
  for (int w = 0; w < 4; ++w) M = fmaxf(M, m_lds[w]);
  const float M_safe = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float wt = fast_exp2(m_lds[w] - M_safe);
    L += wt * l_lds[w], a += wt * o_lds[w][tid];
  }
  if (n_splits == 1) {
    att_out[(int64_t)b * d + h * kHD + tid] = from_float<E>(a / L);
  } else {
    const int64_t pidx = (int64_t)(b * g.n_heads + h) * n_splits + split;
    part_o[pidx * kHD + tid] = a;
    if (tid == 0) part_ml[pidx * 2] = M, part_ml[pidx * 2 + 1] = L;
  }
}

// One workgroup per (query head, sequence), one thread per feature; the splits' loads are requested eight at a time.
template <typename E>
__global__ void __launch_bounds__(128)
    attn_decode_combine_kernel(int n_heads, int n_splits, const float* __restrict__ part_o, const float* __restrict__ part_ml,
                               E* __restrict__ att_out) {
  const int h = blockIdx.x, b = blockIdx.y, f = threadIdx.x;
  const int64_t p0 = (int64_t)(b * n_heads + h) * n_splits;
  float M = -INFINITY, L = 0.f, acc = 0.f;
  constexpr int kTogether = 8;
  for (int s0 = 0; s0 < n_splits; s0 += kTogether) {
    float ms[kTogether], ls[kTogether], v[kTogether];
#pragma unroll
    for (int s = 0; s < kTogether; ++s) {
      const int64_t p = p0 + min(s0 + s, n_splits - 1);
      ms[s] = part_ml[p * 2], ls[s] = part_ml[p * 2 + 1], v[s] = part_o[p * kHD + f];
    }
    float Mg = M;
#pragma unroll
    for (int s = 0; s < kTogether; ++s) Mg = fmaxf(Mg, ms[s]);
    const float r = M == -INFINITY ? 0.f : fast_exp2(M - Mg);
    L *= r, acc *= r;
    M = Mg;
#pragma unroll
    for (int s = 0; s < kTogether; ++s)
      if (s0 + s < n_splits) {
        const float w = ms[s] == -INFINITY ? 0.f : fast_exp2(ms[s] - M);  // (an empty split, possibly before any other)
        L += w * ls[s];
        acc += w * v[s];
      }
  }
  att_out[((int64_t)b * n_heads + h) * kHD + f] = from_float<E>(acc / L);
}

bool attn_decode_supported(int dtype, int tree, const KvGeom& g) {
  return is_16bit(dtype) && g.tiled && g.head_dim == kHD && host_tree(tree)->T == 1;
}

// Key-splits.  A split costs its start, its share of the merge and, the first of them, the merge launch; it is worth the blocks that it takes off
// the others: one up to twelve blocks, then by the square root of the length (at 600 keys 3 splits 59.6 us per layer, 2 62.3).  Beyond about
// three quarters of a workgroup per CU more splits only add up, but for many keys, where a CU with two workgroups of long sequences beside CUs with one
// of short ones is the last to end.  Ungrouped heads are then better off with several workgroups per CU in the other kernel.
// us, steps of 4 layers (the memory-side cache holds the shorter ones' K and V), lengths n / 9 .. n, one split per seven blocks and two workgroups
// per CU / by the square root:
//   32 heads: one sequence of 300 keys 541 / 535, 3000 575 / 565, 6000 620 / 597, 16384 735 / 690; three at 3000 605 / 587, 6000 665 / 641 (two splits
//     685); four at 1000 564 / 557, 3000 626 / 606, 6000 701 / 672; eight at 300 559 / 548, 3000 708 / 677, 6000 870 / 806; twelve at 300 569 / 558,
//     3000 760 / 750; 18 at 3000 883 / 858.  40 heads, 8-bit rows: two at 4000 602 / 598, three 607 / 607 (two splits 636)
//   16 heads: one at 4000 280 / 271, eight at 4000 364 / 345.  8 key/value heads: twelve at 1000 599 / 593, 24 at 300 598 / 584, 1000 626 / 606, 3000
//     718 / 706, 40 at 300 636 / 613, 1000 693 / 682 (at 3000 one split 833, two 821; 24 at 6000 829, three 816)
// Several sequences of ungrouped heads take the other kernel's fewest splits as soon as these are seven blocks long: with K and V from HBM its four
// workgroups per CU ask for more at once.  us, lengths n / 9 .. n, matrix cores / the other kernel, steps of 10 layers: 3 x 32 heads at 900 1009 / 984,
// 1600 1052 / 1010, 2100 1089 / 1022, 5 at 1100 1042 / 1013, 6 at 1100 1073 / 1036, 8 at 900 1073 / 1040 (at 350 976 / 985); 8 layers: 4 x 40 at 1100 1132 / 1102;
// 16 layers: 4 x 16 at 4000 1037 / 997, 5 at 2800 1016 / 976, 10 at 700 984 / 931, 13 at 1100 1013 / 1023; but 2 x 16 (17 splits) at 2800 895 / 926.
// 8-bit rows cost conversions, i.e. vector work: any count of splits pays for them there, and a single sequence takes one workgroup per CU (long ones of 33 heads
// or more the other kernel).  Steps of 3 layers, by the square root / so: 32 heads: one sequence at 5000 329 / 326, three at 900 320 / 312, 2000 331 / 318; 40 heads: four at
// 1300 440 / 425; 16 heads: one at 1300 179 / 176, two at 14000 223 / 210; 8 layers: one of 40 heads at 4000 1121 / 1095, 9000 1206 / 1170 (6 splits 1181).
// Grouped heads: where two workgroups per CU take over.  us, steps of 3 layers, lengths n / 9 .. n, a workgroup per CU / two: 8 key/value heads, 17
// sequences at 2000 350 / 360, 2500 375 / 368, 4000 420 / 407, 18 at 2500 377 / 371, 20 at 3000 400 / 408, 24 at 4000 437 / 447, 16 at 4000 388 / 397; 8-bit rows: 17 at
// 2500 366 / 352, 4000 405 / 362, 24 at 2500 374 / 372, 4000 414 / 393, 28 at 2500 380 / 384, 4000 423 / 417, 12 at 2500 340 / 346, 4000 358 / 353, 10 layers: 7 at 3500
// 1036 / 1049, 20 at 2100 1135 / 1145.
// Few pairs take seven and eight splits early (one sequence at 2000 5 splits 311, 8 307, 16 313), and no more than eight beyond 16 pairs: eight lie on an XCD each
// (steps of 10 layers: 4 sequences at 6000 8 splits 1046, 9 1094, 16 1083, 5 at 8000 8 1110, 10 1124, 12 1159, 3 at 8000 8 1055, 11 1095, 16 1074; but one at 12000
// 8 1082, 12 1048, 16 1045).
// Dealing equal parts of a ragged batch out by its device-side lengths was measured too: 24 sequences of 90 .. 3000 keys
// gain 1 us of 37 (the HBM stream bounds them), a single sequence loses 1 us to finding its part.
static int decode_splits(int B, int kv_heads, int n_heads, int max_prefix, bool q8) {
  const int nb = (max_prefix + 1 + 31) / 32, pairs = B * kv_heads, cus = num_cus();
  int by_len = nb <= 12 ? 1 : (int)sqrtf(0.5f * (float)nb), most;
  const int by_fill = (2 * cus + pairs - 1) / pairs, many = 2 * cus / pairs + 1;  // many: the fewest that the FMA kernel takes
  if (n_heads != kv_heads) {
    // (beyond half as many pairs as CUs, a workgroup per CU leaves no room for a second split)
    const bool few = 2 * pairs <= cus, half = !few && 16 * pairs <= 9 * cus;
    const int fill_from = pairs > cus ? 2048 : q8 ? (few ? 3584 : half ? 2112 : 4 * pairs <= 3 * cus ? 2304 : 3072) : half ? 2304 : 4096;
    most = max_prefix >= fill_from ? by_fill : pairs <= cus ? cus / pairs : 1;
    if (8 * pairs <= cus && nb >= 48 && nb < 128) by_len = nb < 64 ? 7 : 8;
    if (16 * pairs > cus && most > 8) most = 8;
  }
  else if (pairs > cus)
    most = pairs >= 3 * cus ? 1 : max_prefix >= 2048 ? 3 : pairs >= 2 * cus ? 1 : 2;
  else if ((B > 1 ? many <= (q8 ? 32 : 12) : q8 && many <= 16) && (nb + 6) / 7 >= many &&
           max_prefix >= (B == 1 ? 3584 : 4 * pairs <= 3 * cus ? 0 : 640))
    by_len = most = many;
  else if (q8 && B == 1)
    most = cus / pairs, by_len = nb <= 12 ? 1 : (int)sqrtf((float)nb);
  else if (B > 1 && by_len >= many && max_prefix >= 1536)
    most = many;
  else
    most = cus * 3 / 4 / pairs + (B > 1);
  const int s = by_len < most ? by_len : most;
  return s > 32 ? 32 : s < 1 ? 1 : s;
}

// What launch_attention_decode does with a batch.
struct DecodePlan {
  int splits;
  bool fma;      // attn_decode_one_kernel, else attn_decode_kernel
  bool ordered;  // the longest sequences first
};
static DecodePlan decode_plan(const KvGeom& g, int B, int max_prefix) {
  DecodePlan p;
  p.splits = decode_splits(B, g.n_heads, q_heads(g), max_prefix, g.quant != 0);
  const int chunks = (g.group + 31) / 32;
  // Ungrouped heads and more workgroups than the matrix-core kernel keeps resident: FMAs.  (Per layer with small GEMMs, matrix cores /
  // FMAs: 64 sequences x 32 heads of S / 4 .. S keys, S = 16 94.2 / 77.9 us, 100 100.3 / 83.0, 500 149.0 / 140.4, 2000 309.8 / 308.3;
  // 8-bit rows 95.3 / 76.8, 98.4 / 79.0, 124.3 / 105.1, 203.7 / 199.2; 32 at 4000 291.3 / 293.3, 8-bit 185.4 / 183.0.)
  p.fma = g.group == 1 && (int64_t)p.splits * g.n_heads * B > 2 * num_cus();
  // More workgroups than fit at once: long sequences first, from 1536 keys on.  (Finding its place costs a workgroup 1 - 2 us: per layer,
  // lengths S / 4 .. S, in order / not: 64 sequences x 32 heads at S = 100 83.1 / 77.9 us, 500 140.2 / 139.3, 1000 199.3 / 200.1, 2000
  // 309.5 / 313.0; 49 at 2000 246.6 / 256.0; 49 x 8 key/value heads of 4 query heads at 500 77.6 / 73.1, 1000 84.7 / 80.1, 2000 110.9 / 111.2.)
  p.ordered = B > 1 && max_prefix >= 1536 && (int64_t)p.splits * g.n_heads * chunks * B > 2 * num_cus();
  return p;
}

AttentionPlan attn_decode_plan(const KvGeom& g, int B, int max_prefix) {
  const DecodePlan p = decode_plan(g, B, max_prefix);
  return AttentionPlan{p.fma ? ATTN_ONE_FMA : ATTN_ONE_MFMA, 1, p.splits, p.ordered};
}

// (a workspace is sized before the cache's row type is known)
int64_t attn_decode_scratch_bytes(int B, int n_heads, int kv_heads, int max_prefix) {
  const int s16 = decode_splits(B, kv_heads, n_heads, max_prefix, false), s8 = decode_splits(B, kv_heads, n_heads, max_prefix, true);
  const int s = s16 > s8 ? s16 : s8;
  return s == 1 ? 0 : (int64_t)B * n_heads * s * (kHD + 2) * 4;
}

template <typename E, bool Q8>
static int launch_attention_decode_t(const void* q, const Partials* qkv, const float* cs, const KvGeom& g, void* kc, void* vc,
                                     int layer, const int32_t* seq_len, int B, int max_prefix, void* att_out, void* scratch,
                                     int64_t scratch_bytes, hipStream_t st) {
  if (B == 0) return MDZ_OK;
  const DecodePlan plan = decode_plan(g, B, max_prefix);
  const int nq = q_heads(g), splits = plan.splits, chunks = (g.group + 31) / 32;
  MDZ_REQUIRE(scratch_bytes >= attn_decode_scratch_bytes(B, nq, g.n_heads, max_prefix), MDZ_EWORKSPACE,
              "decode attention: scratch too small");
  float* part_o = (float*)scratch;
  float* part_ml = part_o + (int64_t)B * nq * splits * kHD;
  const int cols = g.group < 32 ? g.group : 32;
  const int merge_bytes = 4 * cols * (kORow + 2) * 4, q_bytes = 34 * kQRow;
  const int lds_bytes = merge_bytes > q_bytes ? merge_bytes : q_bytes;
  MDZ_SET_LDS_ONCE((attn_decode_kernel<E, Q8, false>), 4 * 32 * (kORow + 2) * 4);
  MDZ_SET_LDS_ONCE((attn_decode_kernel<E, Q8, true>), 4 * 32 * (kORow + 2) * 4);
  const Partials none = single_slot(nullptr, 0, 0);
  // Non-temporal K and V once a pass reads more of them than the caches hold from one pass to the next.  (us, steps of 4 layers, plain / non-temporal:
  // one sequence x 32 heads at 3000 keys (200 MB) 563 / 568, 6000 610 / 595; 24 x 8 at 300 .. 1000 606 / 620, 3000 (at most 1.2 GB) 719 / 706, 64 x 8 at
  // 1000 (1.1 GB) 735 / 738, 3000 957 / 934, 90 x 8 at 3000 1282 / 1241, but at 500, 6 layers, 1131 / 1142.  More than one key/value head's workgroup per block: plain.)
  const double stream = (double)g.n_layers * B * g.n_heads * max_prefix * (Q8 ? 264 : 512);
  const bool once = chunks == 1 && max_prefix >= 1024 && stream >= (B == 1 ? 350e6 : 640e6);
  if (plan.fma)
    launch_timed(PROF_ATTN, attn_decode_one_kernel<E, Q8>, dim3(splits, g.n_heads, B), 256, 0, st, (const E*)q, qkv ? *qkv : none, cs,
                 g, (E*)kc, (E*)vc, layer, seq_len, max_prefix, (E*)att_out, part_o, part_ml, plan.ordered);
  else
    launch_timed(PROF_ATTN, once ? attn_decode_kernel<E, Q8, true> : attn_decode_kernel<E, Q8, false>, dim3(splits, g.n_heads * chunks, B), 256, lds_bytes, st, (const E*)q,
                 qkv ? *qkv : none, cs, g, (E*)kc, (E*)vc, layer, seq_len, max_prefix, (E*)att_out, part_o, part_ml, plan.ordered);
  MDZ_LAUNCH_CHECK();
  if (splits > 1) {
    launch_timed(PROF_ATTN, attn_decode_combine_kernel<E>, dim3(nq, B), 128, 0, st, nq, splits, part_o, part_ml, (E*)att_out);
    MDZ_LAUNCH_CHECK();
  }
  return MDZ_OK;
}

// qkv: the QKV GEMM's partial sums (RoPE, the cache row and the attention in one kernel), or NULL: q holds rotated queries
int launch_attention_decode(int dtype, const void* q, const Partials* qkv, const float* cs, const KvGeom& g, void* kc, void* vc,
                            int layer, const int32_t* seq_len, int B, int max_prefix, void* att_out, void* scratch,
                            int64_t scratch_bytes, hipStream_t st) {
  if (g.quant)
    MDZ_WITH_ELEM16(dtype, return (launch_attention_decode_t<E, true>(q, qkv, cs, g, kc, vc, layer, seq_len, B, max_prefix,
                                                                      att_out, scratch, scratch_bytes, st)));
  MDZ_WITH_ELEM16(dtype, return (launch_attention_decode_t<E, false>(q, qkv, cs, g, kc, vc, layer, seq_len, B, max_prefix,
                                                                     att_out, scratch, scratch_bytes, st)));
}

}  // namespace mdz
