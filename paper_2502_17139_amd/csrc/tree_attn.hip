// Tree attention of draft trees on gfx950 matrix cores (fc_tree_attention).
//
// The draft tree is verified in one forward pass of the target model
// (Section IV-D, eq. (4)): row i of tree b sits at position prefix_len[b] +
// pos_ids[b][i] and attends to every cached prefix token and to the tree
// rows j with mask[b][i][j] = 1.  This is the layer's attention step for
// those rows, with the rotary embedding of the queries and the tree's keys
// applied by their positions (cached keys are stored rotated).
//
// One workgroup per (tree, query head); one wave per 16 tree rows.  Keys
// and values stream through LDS in blocks of 32 (the cached prefix first,
// then the tree), shared by the workgroup's waves.  Per block a wave
// computes the transposed scores S^T = K Q^T with 16x16x32 bf16 MFMAs (two
// 16-key tiles), applies the mask, updates a running softmax (fp32) and
// accumulates O^T += V^T P^T with eight more MFMAs over the 128 output
// dims.  Working on the transposes keeps every operand in the lane layout
// the MFMA wants: a lane's eight scores are exactly its eight probabilities
// of the value product, so nothing is shuffled between the two products.
//
// The cached prefix moves straight from HBM into LDS with buffer loads that
// write LDS (16 bytes a lane, no registers), through a ring of four blocks,
// so three blocks are in flight while one is used; the loads of rows past
// the prefix fall outside the buffer's range and read as zeros.  Rows sit in
// LDS as written (key-major), each 16-byte chunk XOR-swizzled by the row, so
// the score product reads K rows without bank conflicts and the value
// product takes V^T with the transposing LDS read (ds_read_b64_tr_b16),
// which hands each lane four keys of one output dim.  The tree's own keys
// are rotated on the way in, through registers, up to four blocks at once.
// Workgroups are numbered so that the query heads sharing a key head run on
// the same XCD and its L2 serves their shared key/value reads.
//
// A full batch is bound by HBM (64 trees x 32 heads, 2,048 keys: 490 us, 4.7
// TB/s of keys and values; 510 before the query rows' loads went ahead of
// everything else and the tree's blocks were staged together).  A few trees
// leave CUs idle: their prefixes are cut into parts (split_of), merged by
// k_tree_merge.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fastcoder.h"
#include "fc_device.h"
#include "fc_host.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

constexpr int kD = FC_TREE_ATTN_HEAD_DIM;   // 128
constexpr int kBlock = 32;                  // keys per block
constexpr int kRowBytes = kD * 2;           // 256: one key row
constexpr int kPart = kBlock * kRowBytes;   // 8 KB: a block's keys (or values)
constexpr int kStage = 2 * kPart;           // keys then values
constexpr int kDTiles = kD / 16;            // output tiles of 16 dims
constexpr int kDSteps = kD / 32;            // 32-dim steps of the score product
constexpr int kDmaWaves = 4;                // waves issuing a block's 16 loads, 4 each
constexpr int kXcds = 8;

constexpr int kStages = 4;                  // ring depth
constexpr int kTreeBlocks = 4;              // tree blocks staged at once

// the e-th key of a block that a lane of group lg holds scores of
__device__ __forceinline__ int key_of(int lg, int e) { return e < 4 ? 4 * lg + e : 16 + 4 * lg + (e - 4); }

__device__ __forceinline__ __bf16 f2bf(float x) { return (__bf16)x; }

// byte offset inside a block part of 16-byte chunk c of row r (swizzled)
__device__ __forceinline__ uint32_t chunk_at(int r, int c) { return (uint32_t)(r * kRowBytes + ((c ^ (r & 15)) << 4)); }

// sin and cos of the rotary angle position * freq, freq = base^(-2d/D) of
// the pair (d, d + D/2).  The angle is taken in revolutions and reduced to
// [0, 1) in double precision, so large positions keep full accuracy; the
// hardware sine and cosine then take revolutions directly.
__device__ __forceinline__ void rope_sincos(int pos, double freq, float& s, float& c) {
  constexpr double kInv2Pi = 0.15915494309189533577;
  const double rev = (double)pos * freq * kInv2Pi;
  const float f = (float)(rev - floor(rev));
  s = __builtin_amdgcn_sinf(f);
  c = __builtin_amdgcn_cosf(f);
}

// 8 bf16 as floats.
__device__ __forceinline__ void unpack8(const uint4& u, float (&v)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[2 * e] = __uint_as_float(w[e] << 16);
    v[2 * e + 1] = __uint_as_float(w[e] & 0xFFFF0000u);
  }
}

__device__ __forceinline__ int clamp_len(int len, int most) { return len < 0 ? 0 : (len > most ? most : len); }
__device__ __forceinline__ int prefix_blocks(int P) { return (P + kBlock - 1) / kBlock; }

// kSplit: workgroup blockIdx.y of gridDim.y takes an equal share of the
// prefix's blocks (the last one the tree's rows instead) and leaves its rows'
// running maxima, weight sums and unnormalised outputs in part_ml and part_o
// for k_tree_merge.  A prefix of fewer than split_min blocks stays whole: the
// last workgroup takes all of it, as without kSplit, and the others leave.
template <int MAXT, bool kSplit>
__global__ void __launch_bounds__(MAXT, kSplit && MAXT == 512 ? 2 : 4) k_tree_attn(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_tree, const uint16_t* __restrict__ v_tree,
    const uint16_t* __restrict__ k_cache, const uint16_t* __restrict__ v_cache,
    const int32_t* __restrict__ prefix_len, const int32_t* __restrict__ num_nodes, const int32_t* __restrict__ mask,
    const int32_t* __restrict__ pos_ids, int B, int R, int H, int Hkv, int Pmax, int split_min, double log2_base,
    float* __restrict__ out, float2* __restrict__ part_ml, float* __restrict__ part_o) {
  __shared__ __align__(16) uint8_t s_ring[kStages * kStage];
  __shared__ double s_freq[kD / 2];  // rotary frequencies: one double-precision power per pair and workgroup

  // workgroup -> (tree, head): consecutive ids on one XCD when the count
  // divides evenly, so the heads of one key head share an L2
  const int total = B * H;
  const int x = (int)blockIdx.x;
  const int lin = (total % kXcds == 0) ? (x % kXcds) * (total / kXcds) + x / kXcds : x;
  const int b = lin / H, h = lin - (lin / H) * H;
  const int g_kv = h / (H / Hkv);
  const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
  const int lane = fc::lane_id(), w = __builtin_amdgcn_readfirstlane(tid / fc::kWave);
  const int lg = lane >> 4, lc = lane & 15;  // lane group (0..3), lane column (0..15)
  // this lane's query row, on its way first
  const int qr = w * 16 + lc;
  const bool q_in = qr < R;
  uint4 q_raw[kDSteps];
  int q_pos = 0;
  if (q_in) {
    const uint16_t* src = q + (((int64_t)b * R + qr) * H + h) * kD + 8 * lg;
#pragma unroll
    for (int kc = 0; kc < kDSteps; ++kc) q_raw[kc] = *(const uint4*)(src + 32 * kc);
    q_pos = pos_ids[(int64_t)b * R + qr];
  } else {
#pragma unroll
    for (int kc = 0; kc < kDSteps; ++kc) q_raw[kc] = make_uint4(0u, 0u, 0u, 0u);
  }
  // lengths from the device are clamped to the buffers (a malformed tree,
  // num_nodes = -1, has no rows)
  const int P = clamp_len(prefix_len[b], Pmax);
  const int n_all = prefix_blocks(P);
  const int part = kSplit ? (int)blockIdx.y : 0, parts = kSplit ? (int)gridDim.y - 1 : 1;
  const bool whole = !kSplit || n_all < split_min;
  if (whole && part < (kSplit ? parts : 0)) return;
  const int n = clamp_len(num_nodes[b], R);
  const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)s_ring;

  // this workgroup's prefix blocks [blk0, n_pre) and tree blocks
  const int blk0 = whole ? 0 : (int)((uint32_t)n_all * (uint32_t)part / (uint32_t)parts);  // n_all < 2^26
  const int n_pre = whole ? n_all
                    : part < parts ? (int)((uint32_t)n_all * (uint32_t)(part + 1) / (uint32_t)parts) : blk0;
  const int n_tree = whole || part == parts ? (n + kBlock - 1) / kBlock : 0;
  const int key_end = P < n_pre * kBlock ? P : n_pre * kBlock;

  // Prefix block loads: load u (0..15) of a block covers rows 4(u%8) ..
  // 4(u%8)+3 of the keys (u < 8) or values; lane L takes row 4(u%8) + L/16
  // and fills physical chunk L%16, i.e. logical chunk (L%16) ^ (row%16).
  // Waves 0..3 issue loads w, w+4, w+8, w+12 of every block.
  const int64_t row_stride = (int64_t)Hkv * kD * 2;  // bytes between consecutive keys
  const uint32_t pre_bytes = P > 0 ? (uint32_t)((int64_t)(P - 1) * row_stride + kRowBytes) : 0u;
  const fc::int32x4 rk = fc::buffer_rsrc(k_cache + ((int64_t)b * Pmax * Hkv + g_kv) * kD, pre_bytes);
  const fc::int32x4 rv = fc::buffer_rsrc(v_cache + ((int64_t)b * Pmax * Hkv + g_kv) * kD, pre_bytes);
  const bool dma_wave = w < kDmaWaves;
  auto issue_block = [&](int blk) {  // rows past key_end (also whole blocks) read as zeros, from no memory
    if (!dma_wave) return;
    const uint32_t slot = ring + (uint32_t)((blk % kStages) * kStage);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = w + kDmaWaves * i;
      const int r = 4 * (u & 7) + (lane >> 4);
      const int c = (lane & 15) ^ (r & 15);
      const int64_t key = (int64_t)blk * kBlock + r;
      const uint32_t voff = key < key_end ? (uint32_t)(key * row_stride + 16 * c) : pre_bytes;
      fc::lds_load16(slot + (u < 8 ? 0u : (uint32_t)kPart) + (uint32_t)(u & 7) * 1024u, voff, u < 8 ? rk : rv);
    }
  };

  for (int d = tid; d < kD / 2; d += nt) s_freq[d] = exp2(-2.0 * (double)d / (double)kD * log2_base);

  // the first prefix blocks on their way
#pragma unroll
  for (int u = 0; u < kStages - 1; ++u) issue_block(blk0 + u);
  // the frequencies are in LDS; the loads in flight are not waited for
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  // the query row's rotated dims as the B operand of S^T
  bf16x8 qf[kDSteps];
  {
    float v[kDSteps][8];
#pragma unroll
    for (int kc = 0; kc < kDSteps; ++kc) unpack8(q_raw[kc], v[kc]);
    const int pos = P + q_pos;
#pragma unroll
    for (int kc = 0; kc < kDSteps / 2; ++kc)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        // dims d and d + D/2 sit in steps kc and kc + 2 of the same lane
        float s, c;
        rope_sincos(pos, s_freq[32 * kc + 8 * lg + e], s, c);
        const float x0 = v[kc][e], x1 = v[kc + 2][e];
        v[kc][e] = x0 * c - x1 * s;
        v[kc + 2][e] = x1 * c + x0 * s;
      }
#pragma unroll
    for (int kc = 0; kc < kDSteps; ++kc)
#pragma unroll
      for (int e = 0; e < 8; ++e) qf[kc][e] = f2bf(v[kc][e]);
  }

  floatx4 o[kDTiles];
#pragma unroll
  for (int t = 0; t < kDTiles; ++t) o[t] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  float m_run = -INFINITY, l_run = 0.0f;
  const float scale = 1.0f / sqrtf((float)kD);

  // One block of the two products from the K and V parts at slot_off (a byte
  // offset in s_ring); bit e of `allow` admits this lane's e-th key.
  auto consume = [&](uint32_t slot_off, uint32_t allow) {
    const uint8_t* sk = s_ring + slot_off;
    floatx4 st0 = {0.0f, 0.0f, 0.0f, 0.0f}, st1 = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int kc = 0; kc < kDSteps; ++kc) {
      const bf16x8 a0 = *(const bf16x8*)(sk + chunk_at(lc, 4 * kc + lg));
      const bf16x8 a1 = *(const bf16x8*)(sk + chunk_at(16 + lc, 4 * kc + lg));
      st0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, qf[kc], st0, 0, 0, 0);
      st1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, qf[kc], st1, 0, 0, 0);
    }
    // this lane holds keys 4*lg + i and 16 + 4*lg + i for query row qr
    float sv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const bool ok = (allow >> e) & 1u;
      const float raw = e < 4 ? st0[e] : st1[e - 4];
      sv[e] = ok ? raw * scale : -INFINITY;
    }
    float mb = sv[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) mb = fmaxf(mb, sv[e]);
    mb = fmaxf(mb, __shfl_xor(mb, 16));
    mb = fmaxf(mb, __shfl_xor(mb, 32));
    const float m_new = fmaxf(m_run, mb);
    const bool none = m_new == -INFINITY;  // no allowed key for this row yet
    const float alpha = none ? 1.0f : __expf(m_run - m_new);
    bf16x8 pb;
    float ps = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float pe = none ? 0.0f : __expf(sv[e] - m_new);
      ps += pe;
      pb[e] = f2bf(pe);
    }
    m_run = m_new;
    l_run = l_run * alpha + ps;
    // V^T for output tile t: a transposing read gives lane (lg, lc) dims
    // 16t + lc of keys 4lg + e (first read) and 16 + 4lg + e (second); the
    // addressing lane (lg, 4e + i) points at dims 16t + 4i of that key
    const uint32_t vbase = ring + slot_off + (uint32_t)kPart;
    const int vr0 = 4 * lg + (lc >> 2), vr1 = 16 + 4 * lg + (lc >> 2), vq = lc & 3;
#pragma unroll
    for (int t = 0; t < kDTiles; ++t) {
      o[t] *= alpha;
      const int cc = 2 * t + (vq >> 1);
      const uint32_t half = (uint32_t)(vq & 1) * 8u;
      const bf16x4 lo4 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (lds_bf16x4*)(uintptr_t)(vbase + chunk_at(vr0, cc) + half));
      const bf16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
          (lds_bf16x4*)(uintptr_t)(vbase + chunk_at(vr1, cc) + half));
      const bf16x8 a = {lo4[0], lo4[1], lo4[2], lo4[3], hi4[0], hi4[1], hi4[2], hi4[3]};
      o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pb, o[t], 0, 0, 0);
    }
  };

  // the cached prefix: a ring of kStages blocks, kStages - 1 in flight
  for (int blk = blk0; blk < n_pre; ++blk) {
    // this wave's loads of block blk are done once at most the loads of the
    // kStages - 2 later blocks (4 each) are outstanding; the barrier makes every
    // wave's visible, and frees the slot the next issue overwrites
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * (kStages - 2)) : "memory");
    __syncthreads();
    issue_block(blk + kStages - 1);
    uint32_t allow = q_in ? 0xFFu : 0u;
    if (blk == n_all - 1) {  // the prefix may end inside the block
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (blk * kBlock + key_of(lg, e) >= P) allow &= ~(1u << e);
    }
    consume((uint32_t)((blk % kStages) * kStage), allow);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  // the tree's rows: keys rotated by their positions, values as they are,
  // through registers into the ring, kTreeBlocks blocks at a time, so that
  // their loads and the mask's are waited for once
  constexpr int kMaskUnroll = kSplit && MAXT == 512 ? kTreeBlocks : 1;  // one part: two workgroups share the registers
  for (int tb0 = 0; tb0 < n_tree; tb0 += kTreeBlocks) {
    const int nb = n_tree - tb0 < kTreeBlocks ? n_tree - tb0 : kTreeBlocks;
    uint32_t allow = 0;  // eight bits per block
#pragma unroll kMaskUnroll
    for (int u = 0; u < nb; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int j = (tb0 + u) * kBlock + key_of(lg, e);
        if (j < n && qr < n && mask[((int64_t)b * R + qr) * R + j] == 1) allow |= 1u << (8 * u + e);
      }
    for (int it = tid; it < nb * kBlock * (kD / 16); it += nt) {
      const int row = it / (kD / 16), c = it - row * (kD / 16);  // key, chunks c and c + D/16
      const int j = tb0 * kBlock + row;
      uint8_t* sk = s_ring + (row / kBlock) * kStage;
      float a[8], bb[8];
      uint4 k0 = make_uint4(0u, 0u, 0u, 0u), k1 = k0, v0 = k0, v1 = k0;
      if (j < n) {
        const int64_t src = (((int64_t)b * R + j) * Hkv + g_kv) * kD;
        k0 = *(const uint4*)(k_tree + src + 8 * c);
        k1 = *(const uint4*)(k_tree + src + kD / 2 + 8 * c);
        v0 = *(const uint4*)(v_tree + src + 8 * c);
        v1 = *(const uint4*)(v_tree + src + kD / 2 + 8 * c);
        const int pos = P + pos_ids[(int64_t)b * R + j];
        unpack8(k0, a);
        unpack8(k1, bb);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float sn, cs;
          rope_sincos(pos, s_freq[8 * c + e], sn, cs);
          const float x0 = a[e], x1 = bb[e];
          a[e] = x0 * cs - x1 * sn;
          bb[e] = x1 * cs + x0 * sn;
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = bb[e] = 0.0f;
      }
      bf16x8 pa, pbb;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pa[e] = f2bf(a[e]);
        pbb[e] = f2bf(bb[e]);
      }
      const int kk = row % kBlock;
      *(bf16x8*)(sk + chunk_at(kk, c)) = pa;
      *(bf16x8*)(sk + chunk_at(kk, c + kD / 16)) = pbb;
      *(uint4*)(sk + kPart + chunk_at(kk, c)) = v0;
      *(uint4*)(sk + kPart + chunk_at(kk, c + kD / 16)) = v1;
    }
    __syncthreads();
    for (int u = 0; u < nb; ++u) consume((uint32_t)(u * kStage), (allow >> (8 * u)) & 0xFFu);
    __syncthreads();
  }

  // normalise by the row's total weight (summed over the four lane groups)
  float lt = l_run + __shfl_xor(l_run, 16);
  lt = lt + __shfl_xor(lt, 32);
  if (!whole) {
    if (q_in) {
      const int64_t row = ((int64_t)(b * H + h) * gridDim.y + blockIdx.y) * R + qr;
      if (lg == 0) part_ml[row] = make_float2(m_run, lt);
#pragma unroll
      for (int t = 0; t < kDTiles; ++t) *(floatx4*)(part_o + row * kD + 16 * t + 4 * lg) = o[t];
    }
    return;
  }
  if (q_in) {
    const bool live = qr < n && lt > 0.0f;
    const float inv = live ? 1.0f / lt : 0.0f;
    float* dst = out + (((int64_t)b * R + qr) * H + h) * kD;
#pragma unroll
    for (int t = 0; t < kDTiles; ++t) {
      floatx4 r = o[t] * inv;
      *(floatx4*)(dst + 16 * t + 4 * lg) = r;
    }
  }
}

// The parts of a split row put together: out = sum_s e^(m_s - m) o_s / sum_s
// e^(m_s - m) l_s with m the largest m_s.  32 lanes per (row, head), four dims
// each, every part's loads issued before any is used; a row at or past
// num_nodes[b] is 0.  A whole prefix's rows are in place already.
template <int kMost>
__global__ void __launch_bounds__(256) k_tree_merge(const float2* __restrict__ part_ml,
                                                      const float* __restrict__ part_o,
                                                      const int32_t* __restrict__ prefix_len,
                                                      const int32_t* __restrict__ num_nodes, int R, int H, int Pmax,
                                                      int split_min, int parts, float* __restrict__ out) {
  const int b = (int)blockIdx.y;
  const int i = (int)((blockIdx.x * 256 + threadIdx.x) >> 5);  // (row, h)
  if (i >= R * H) return;
  const int d = 4 * (int)(threadIdx.x & 31);
  const int h = i % H, qr = i / H;
  if (prefix_blocks(clamp_len(prefix_len[b], Pmax)) < split_min) return;
  const int64_t row0 = (int64_t)(b * H + h) * parts * R + qr;
  float2 ml[kMost];
  floatx4 o[kMost];
#pragma unroll
  for (int s = 0; s < kMost; ++s) {
    ml[s] = s < parts ? part_ml[row0 + (int64_t)s * R] : make_float2(-INFINITY, 0.0f);
    o[s] = s < parts ? *(const floatx4*)(part_o + (row0 + (int64_t)s * R) * kD + d) : floatx4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  float m = -INFINITY;
#pragma unroll
  for (int s = 0; s < kMost; ++s) m = fmaxf(m, ml[s].x);
  floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  float l = 0.0f;
#pragma unroll
  for (int s = 0; s < kMost; ++s) {
    const float w = ml[s].x > -INFINITY ? __expf(ml[s].x - m) : 0.0f;  // 0 for a part without an allowed key
    l += w * ml[s].y;
    acc += w * o[s];
  }
  acc *= qr < num_nodes[b] && l > 0.0f ? 1.0f / l : 0.0f;
  *(floatx4*)(out + ((int64_t)b * R * H + i) * kD + d) = acc;
}

// How a call splits: workgroups per (tree, head) - 1, or `parts` - 1 for the
// prefix and one for the tree's rows - and the blocks from which a prefix is
// cut.  A workgroup walks its prefix at about 1 us per block of 32 keys (a
// chain of LDS reads, products and a softmax step), so with few (tree, head)
// pairs most of the chip idles while that chain runs; against it stand the
// parts' rows written and read again, which grow with the tree's rows.
// Measured against one part (us, two figures: one part -> split):
//  - up to a workgroup per CU in all (85 pairs): 1 tree x 32 heads, 65 rows:
//    3,000 keys 92 -> 24.7 in 8 parts (50 in 3, 31 in 5, 35 in 10), 320 keys
//    19.8 -> 17.8, 192 keys 16.4 -> 17.5; 129 rows: 512 keys 36.0 -> 33.8, 320
//    keys 29.7 -> 32.2; 256 rows: 384 keys 66.5 -> 65.2.
//  - 86 to 128 pairs, in three parts: the prefixes have a CU per workgroup, the
//    trees share one.  128 pairs, 65 rows: 2,048 keys 70.9 -> 50.9, 768 keys 34.8
//    -> 32.6, 512 keys 28.1 -> 29.1; 17 rows: 512 keys 18.9 -> 14.9; 256 rows:
//    1,536 keys 118 -> 110, 1,024 keys 96.5 -> 97.8.
//  - 129 to 170 pairs, in three parts: the prefixes share CUs too, and only
//    trees of up to 64 rows (four waves) gain.  160 pairs, 49 rows: 1,024 keys
//    33.1 -> 29.2, 512 keys 22.2 -> 21.1; 65 rows: 39.5 -> 45.6 and 4,096 keys
//    131.5 -> 132.3.
// With more, 256 pairs 73 -> 87.  A call is launched in parts where its buffer
// could hold a prefix long enough, and each tree is cut by its own prefix: the
// lengths are on the device.  A tree left whole there takes 1 to 2 us more than
// in a call of one part (the merge's launch): 32 pairs, 65 rows, no prefix 10.7
// -> 11.8.
constexpr int kCus = 256;
constexpr int kMaxParts = 16;
struct Split {
  int parts, min_blocks;
};
Split split_of(int32_t B, int32_t R, int32_t H, int32_t Pmax) {
  const int64_t wgs = (int64_t)B * H, blocks = ((int64_t)Pmax + kBlock - 1) / kBlock;
  const bool fits = 3 * wgs <= kCus;  // a workgroup per CU in three parts
  const int least = fits ? (R < 32 ? 6 : R < 128 ? 4 + R / 16 : 12) : 16 + R / 10;
  if (blocks < least) return {1, 0};
  if (!fits && 2 * wgs > kCus && (R > 64 || 3 * wgs > 2 * kCus)) return {1, 0};
  int64_t parts = fits ? kCus / wgs : 3;
  if (parts > kMaxParts) parts = kMaxParts;
  if (parts > blocks / 2 + 1) parts = blocks / 2 + 1;  // two blocks or more each
  return {(int)parts, least};
}

size_t carve_parts(void* p, int32_t B, int32_t R, int32_t H, int parts, float2** ml, float** o) {
  fc::Carver c(p);
  const size_t rows = (size_t)B * H * parts * R;
  *ml = c.take<float2>(rows);
  *o = c.take<float>(rows * kD);
  return c.used + 256;
}

}  // namespace

extern "C" size_t fc_tree_attention_workspace_bytes(int32_t B, int32_t R, int32_t H, int32_t Pmax) {
  if (B < 1 || R < 1 || R > FC_MAX_TREE_ROWS || H < 1 || Pmax < 0) return 0;
  const int parts = split_of(B, R, H, Pmax).parts;
  float2* ml;
  float* o;
  return parts > 1 ? carve_parts(nullptr, B, R, H, parts, &ml, &o) : 0;
}

extern "C" fc_status fc_tree_attention(const uint16_t* q, const uint16_t* k_tree, const uint16_t* v_tree,
                                       const uint16_t* k_cache, const uint16_t* v_cache, const int32_t* prefix_len,
                                       const int32_t* num_nodes, const int32_t* mask, const int32_t* pos_ids,
                                       int32_t B, int32_t R, int32_t H, int32_t Hkv, int32_t D, int32_t Pmax,
                                       float rope_base, float* out, hipStream_t stream) {
  return fc_tree_attention_ws(q, k_tree, v_tree, k_cache, v_cache, prefix_len, num_nodes, mask, pos_ids, B, R, H, Hkv,
                              D, Pmax, rope_base, out, nullptr, 0, stream);
}

extern "C" fc_status fc_tree_attention_ws(const uint16_t* q, const uint16_t* k_tree, const uint16_t* v_tree,
                                       const uint16_t* k_cache, const uint16_t* v_cache, const int32_t* prefix_len,
                                       const int32_t* num_nodes, const int32_t* mask, const int32_t* pos_ids,
                                       int32_t B, int32_t R, int32_t H, int32_t Hkv, int32_t D, int32_t Pmax,
                                       float rope_base, float* out, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (B < 0 || R < 1 || R > FC_MAX_TREE_ROWS || H < 1 || Hkv < 1 || H % Hkv != 0 || Pmax < 0) return FC_ERR_INVALID;
  if (!(rope_base > 1.0f)) return FC_ERR_INVALID;
  if (D != FC_TREE_ATTN_HEAD_DIM) return FC_ERR_UNSUPPORTED;
  if (B == 0) return FC_OK;
  if (!q || !k_tree || !v_tree || !prefix_len || !num_nodes || !mask || !pos_ids || !out) return FC_ERR_INVALID;
  if (Pmax > 0 && (!k_cache || !v_cache)) return FC_ERR_INVALID;
  const uintptr_t al = (uintptr_t)q | (uintptr_t)k_tree | (uintptr_t)v_tree | (uintptr_t)out |
                       (Pmax > 0 ? ((uintptr_t)k_cache | (uintptr_t)v_cache) : 0);
  if (al & 15) return FC_ERR_INVALID;
  // the prefix of one (tree, key head) is read with 32-bit byte offsets
  if ((int64_t)Pmax * Hkv * D * 2 >= (int64_t)1 << 32) return FC_ERR_UNSUPPORTED;
  const int rows_waves = (R + 15) / 16;
  const int waves = rows_waves < 4 ? 4 : rows_waves;  // at least 256 threads stage a block
  const Split sp = split_of(B, R, H, Pmax);
  int parts = sp.parts;
  float2* ml = nullptr;
  float* po = nullptr;
  if (parts > 1) {
    if (!ws || ws_bytes < fc_tree_attention_workspace_bytes(B, R, H, Pmax)) {
      parts = 1;
    } else {
      if ((uintptr_t)ws & 15) return FC_ERR_INVALID;
      carve_parts(ws, B, R, H, parts, &ml, &po);
    }
  }
  const dim3 grid((uint32_t)B * (uint32_t)H, (uint32_t)parts), block(waves * fc::kWave);
  (void)hipGetLastError();
#define FC_ATTN(T, SPLIT)                                                                                              \
  hipLaunchKernelGGL((k_tree_attn<T, SPLIT>), grid, block, 0, stream, q, k_tree, v_tree, k_cache, v_cache, prefix_len, \
                     num_nodes, mask, pos_ids, B, R, H, Hkv, Pmax, sp.min_blocks, log2((double)rope_base), out, ml, po)
  // trees of up to 128 rows (c <= 127) in workgroups of at most 8 waves,
  // which leaves each lane the registers the accumulators need
  if (waves <= 8 && parts == 1) FC_ATTN(512, false);
  else if (waves <= 8) FC_ATTN(512, true);
  else if (parts == 1) FC_ATTN(1024, false);
  else FC_ATTN(1024, true);
#undef FC_ATTN
  FC_CHECK_LAUNCH();
  if (parts > 1) {
    auto merge = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(fc::div_up((uint64_t)R * H * 32, 256), B), dim3(256), 0, stream, ml, po,
                         prefix_len, num_nodes, R, H, Pmax, sp.min_blocks, parts, out);
    };
    if (parts <= 4)
      merge(k_tree_merge<4>);
    else if (parts <= 8)
      merge(k_tree_merge<8>);
    else
      merge(k_tree_merge<kMaxParts>);
    FC_CHECK_LAUNCH();
  }
  return FC_OK;
}
