// Causal GQA prefill attention of the computed rows over the assembled KV
// (Section 5.3, "Completing prefill": the recompute ranges and the remaining
// prompt are processed in one extend pass).
//
// Row t at prompt position p_t, query head h, KV head g = h / G:
//   o = softmax(scale * q_rot . K[0..p_t, g]^T) V[0..p_t, g]
// with q_rot = RoPE(q, p_t) rounded to the activation dtype and keys visible
// up to and including p_t.
//
// Three kernels:
//   attn_f32_kernel   fp32 reference mode, fp64 MFMA, one workgroup per 16
//                     rows and query head.
//   attn_mfma_kernel  bf16 mode.  Work item = R row blocks of up to 32
//                     rows of one request x one KV head (R = 1 or 3, chosen
//                     per plan), consecutive in the plan's item row order
//                     (AttnRow: with R = 3 the rows of each request grouped
//                     by first visible key); the query heads of that
//                     KV head are packed into the workgroup (four waves per
//                     row block, one head each; G = 8 takes two items), so
//                     every K/V tile staged in LDS feeds all of them.  Per
//                     32-key tile (K loaded straight into
//                     LDS, V staged through registers as V^T in fp16):
//                       S^T = K Q^T        v_mfma_f32_32x32x16_bf16
//                       online softmax     fp32, exp2 with folded scale;
//                                          the running max moves only when
//                                          a tile's probability sum says so
//                       O^T += V^T P^T     v_mfma_f32_32x32x16_f16
//                     Keeping S and O transposed gives every lane one query
//                     row, so row statistics are lane-local except for one
//                     exchange between the two half-waves.  P and V enter the
//                     second product as fp16 (bf16 P would cost ~2e-3
//                     relative error; fp16 keeps it near 2e-4).  A wave
//                     holds at most 168 registers, so three waves share each
//                     SIMD.  LDS per workgroup: 36 KB of K/V tiles plus
//                     16.5 KB of cos/sin rows per row block, 52.5 KB with
//                     one row block (three 4-wave workgroups per CU) and
//                     85.5 KB with three (one 12-wave workgroup per CU).
//                     An item whose key range the plan split writes its
//                     normalized rows and log-sum-exp in fp32 instead (one
//                     split buffer slot per row block).
//   attn_merge_kernel merges the key ranges of split items into out, lse.
#include <cmath>
#include <type_traits>

#include "attn_common.h"
#include "kernels_common.h"
#include "tsr_internal.h"

namespace tsr {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------- fp32 mode
// The reference mode of the fp32 configurations: operands are fp32 (q_rot
// and K rounded to fp32 like the storage), the arithmetic is fp64 (scores,
// softmax statistics and the weighted sum of V), and the output is rounded
// to fp32 once.
//
// Bound by latency: these batches are a few hundred rows (the tiny
// configuration's whole launch is 20 MFLOP), so the work is cut for
// parallelism.  A workgroup takes 16 rows of one query head; its waves take
// the 16-key tiles of the rows' key range in turn, each with its own running
// softmax, merged through LDS at the end.  Both products run on
// v_mfma_f64_16x16x4_f64:
//   S^T = K Q^T   lane l holds key l % 16 and row l % 16 over the D/4
//                 consecutive dims of quarter l / 16 (the order of the
//                 contraction is free, so a lane's dims are whole 16-byte
//                 loads of its row);
//   O^T += V^T P^T  result register r of S^T is key 4 r + l / 16 of the
//                 tile, which is the operand layout of step r: P needs no
//                 exchange.
// 272 prompt tokens, 152 rows, 4 heads of 64: 1,176 us with scalar code, one
// workgroup per 32 rows and KV head, rows one after another; 20 us so.
typedef double f64x4 __attribute__((ext_vector_type(4)));

// Waves of a workgroup: eight, and four at head_dim 256, where a wave's
// output tile alone is 128 registers (28 registers spill there, at one wave a
// SIMD; three requests, 360 rows, 4 heads of 256: 4,059 us with the scalar
// code, 204 so).
template <int D> constexpr int kF32Waves = D == 256 ? 4 : 8;
constexpr int kF32Rows = 16, kF32Keys = 16;

template <int D>
__global__ __launch_bounds__(64 * kF32Waves<D>) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ kc,
    const float* __restrict__ vc, const AttnItem* __restrict__ items,
    const int32_t* __restrict__ bts, const RowDesc* __restrict__ rows,
    const float* __restrict__ rope_cos, const float* __restrict__ rope_sin,
    float* __restrict__ out, float* __restrict__ lse, int n_q_heads,
    int n_kv_heads, int log2_page, float scale) {
  constexpr int NW = kF32Waves<D>;
  constexpr int DQ = D / 4;      // dims of a lane in S^T = K Q^T
  constexpr int DT = D / 16;     // 16-dim blocks of the output
  constexpr int kRound = 4;      // 16-dim blocks merged per round
  __shared__ double om[NW][16 * kRound][kF32Rows];
  __shared__ double ml[2][NW][kF32Rows];
  const AttnItem it = items[blockIdx.x];
  const int r0 = kF32Rows * blockIdx.z;
  if (r0 >= it.n_rows) return;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = tid & 15, c4 = (tid >> 4) & 3;
  const int G = n_q_heads / n_kv_heads;
  const int g = it.kv_head;
  const int hq = g * G + blockIdx.y;
  const int page_mask = (1 << log2_page) - 1;
  const int32_t* bt = bts + it.bt_off;
  // rows past the item's last one repeat it and store nothing
  const int n_rows = min(kF32Rows, it.n_rows - r0);
  const int row = it.row0 + r0 + min(c16, n_rows - 1);
  const int pos = rows[row].pos;
  // positions ascend
  const int min_pos = rows[it.row0 + r0].pos;
  const int kv_end = rows[it.row0 + r0 + n_rows - 1].pos + 1;

  // this lane's dims of the rotated query
  float qr[DQ];
  {
    constexpr int H = D / 2;
    const int d0 = DQ * c4, dl = d0 % H;   // first dim, and its index in a RoPE half
    const float* qp = q + ((int64_t)row * n_q_heads + hq) * D + dl;
    const float* cp = rope_cos + (int64_t)pos * H + dl;
    const float* sp = rope_sin + (int64_t)pos * H + dl;
#pragma unroll
    for (int e = 0; e < DQ; e += 4) {
      const float4 a = *reinterpret_cast<const float4*>(qp + e);
      const float4 b = *reinterpret_cast<const float4*>(qp + H + e);
      const float4 c = *reinterpret_cast<const float4*>(cp + e);
      const float4 s = *reinterpret_cast<const float4*>(sp + e);
      float lo[4] = {a.x, a.y, a.z, a.w}, hi[4] = {b.x, b.y, b.z, b.w};
      const float cs[4] = {c.x, c.y, c.z, c.w}, sn[4] = {s.x, s.y, s.z, s.w};
      rope_rotate<4>(lo, hi, cs, sn);
#pragma unroll
      for (int i = 0; i < 4; ++i) qr[e + i] = d0 < H ? lo[i] : hi[i];
    }
  }

  f64x4 o[DT];
#pragma unroll
  for (int t = 0; t < DT; ++t) o[t] = f64x4{0.0, 0.0, 0.0, 0.0};
  double m = -INFINITY, l = 0.0;
  const double sc = scale;
  auto key_base = [&](int k) -> int64_t {   // keys past the range read its last one
    const int kk = min(k, kv_end - 1);
    return ((((int64_t)bt[kk >> log2_page] * n_kv_heads + g) << log2_page) + (kk & page_mask)) * D;
  };
  for (int k0 = it.kv_lo + kF32Keys * w; k0 < kv_end; k0 += kF32Keys * NW) {
    const float* kp = kc + key_base(k0 + c16) + DQ * c4;
    float4 kr[DQ / 4];
#pragma unroll
    for (int e = 0; e < DQ / 4; ++e) kr[e] = *reinterpret_cast<const float4*>(kp + 4 * e);
    const float* vp[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) vp[r] = vc + key_base(k0 + 4 * r + c4) + c16;
    f64x4 s = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < DQ / 4; ++e) {
      s = __builtin_amdgcn_mfma_f64_16x16x4f64(kr[e].x, qr[4 * e], s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f64_16x16x4f64(kr[e].y, qr[4 * e + 1], s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f64_16x16x4f64(kr[e].z, qr[4 * e + 2], s, 0, 0, 0);
      s = __builtin_amdgcn_mfma_f64_16x16x4f64(kr[e].w, qr[4 * e + 3], s, 0, 0, 0);
    }
    // register r of row c16: key k0 + 4 r + c4
    double mt = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = k0 + 4 * r + c4 <= pos ? s[r] * sc : -INFINITY;
      mt = fmax(mt, s[r]);
    }
    mt = fmax(mt, __shfl_xor(mt, 16));
    mt = fmax(mt, __shfl_xor(mt, 32));
    const double mn = fmax(m, mt);
    // a row that sees no key of the wave's tiles yet keeps m at -inf
    const double mb = mn == -INFINITY ? 0.0 : mn;
    const double alpha = exp(m - mb);
    m = mn;
    double p[4], ps = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p[r] = exp(s[r] - mb);
      ps += p[r];
    }
    l = l * alpha + ps;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[t][i] *= alpha;
    // A row must not meet the V of keys past its own: they weigh 0, but
    // 0 x inf is not 0.  Only tiles past the block's smallest position hold
    // such keys; if a V there is not finite, each row sums its own keys.
    bool plain = true;
    if (k0 + kF32Keys - 1 > min_pos) {
      float z = 0.0f;
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (k0 + 4 * r + c4 < kv_end)
#pragma unroll
          for (int t = 0; t < DT; ++t) z = fmaf(vp[r][16 * t], 0.0f, z);
      plain = __builtin_amdgcn_ballot_w64(z != 0.0f) == 0;
    }
    if (plain) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool in = k0 + 4 * r + c4 < kv_end;
#pragma unroll
        for (int t = 0; t < DT; ++t)
          o[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? (double)vp[r][16 * t] : 0.0, p[r],
                                                      o[t], 0, 0, 0);
      }
    } else {
#pragma unroll 1
      for (int j = 0; j < kF32Keys; ++j) {
        const double pr = j < 8 ? (j < 4 ? p[0] : p[1]) : (j < 12 ? p[2] : p[3]);
        const double pj = __shfl(pr, 16 * (j % 4) + c16);
        if (k0 + j > pos) continue;
        const float* vj = vc + key_base(k0 + j) + c4;
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) o[t][i] = fma(pj, (double)vj[16 * t + 4 * i], o[t][i]);
      }
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  // merge the waves: weights exp(m_w - M), M the row's maximum (every row
  // sees a key, so M is finite)
  if (c4 == 0) {
    ml[0][w][c16] = m;
    ml[1][w][c16] = l;
  }
  __syncthreads();
  double M = -INFINITY, L = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) M = fmax(M, ml[0][i][c16]);
#pragma unroll
  for (int i = 0; i < NW; ++i) L += ml[1][i][c16] * exp(ml[0][i][c16] - M);
  const double wt = exp(m - M) / L;
  for (int t0 = 0; t0 < DT; t0 += kRound) {
    if (t0) __syncthreads();
#pragma unroll
    for (int t = 0; t < DT; ++t)
      if (t / kRound * kRound == t0)
#pragma unroll
        for (int r = 0; r < 4; ++r) om[w][16 * (t - t0) + 4 * r + c4][c16] = o[t][r] * wt;
    __syncthreads();
    for (int i = tid; i < 16 * kRound * kF32Rows; i += 64 * NW) {
      const int d = i % (16 * kRound), r = i / (16 * kRound);
      double a = 0.0;
#pragma unroll
      for (int x = 0; x < NW; ++x) a += om[x][d][r];
      if (r < n_rows)
        out[((int64_t)(it.row0 + r0 + r) * n_q_heads + hq) * D + 16 * t0 + d] = (float)a;
    }
  }
  if (lse && w == 0 && c4 == 0 && c16 < n_rows)
    lse[(int64_t)row * n_q_heads + hq] = (float)(M + log(L));
}

// ------------------------------------------------------------- bf16 mode
__device__ __forceinline__ uint32_t pack_f16x2(float a, float b) {
  // bf16 values convert to fp16 exactly inside fp16's normal range (the
  // largest bf16 below fp16's maximum is 65280); a larger one becomes
  // infinite, so outputs that read it are non-finite instead of clipped.
  const f16x2 h = {(_Float16)a, (_Float16)b};
  return __builtin_bit_cast(uint32_t, h);
}
// A K tile in LDS: for each 16-key block, four 1 KB blocks of 32 dims, in
// which 8-dim chunk c of key k lies at 256 c + 16 k.  Fragment reads are
// 256-byte runs at immediate offsets, and a direct load of 16 bytes a lane
// by a wave that reads one page fills a 1 KB block.
constexpr int kKHalf = 4 * kKBlk;

// Masking of a tile's scores (tile loops are instantiated per kind).
constexpr int kNoMask = 0, kMaskCausal = 1, kMaskBoth = 2;
using NoMask = std::integral_constant<int, kNoMask>;
using MaskCausal = std::integral_constant<int, kMaskCausal>;
using MaskBoth = std::integral_constant<int, kMaskBoth>;

// AV: V aliasing -- the V of a 16-key block comes from the page the V block
// table names, a pool page when kPoolPageFlag is set (else the request page
// the K block table names).
// AK: K rotated on load -- the K of a 16-key block comes from the page the K
// block table names; a pool page (kPoolPageFlag) holds the cached keys before
// RoPE, which the staging waves rotate at the keys' positions (fp32 table,
// no fused multiply-add, bf16 rounding: the arithmetic of compose) and write
// to LDS in fragment order.
// R: row blocks per workgroup.  Waves 4 b .. 4 b + 3 own the 32 rows of row
// block b; the first four waves stage every K/V tile for all of them.
template <int G, bool AV, bool AK, int R>
__global__ __launch_bounds__(256 * R, 3) void attn_mfma_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kc,
    const uint16_t* __restrict__ vc, const uint16_t* __restrict__ pool_k,
    const uint16_t* __restrict__ pool_v,
    const AttnItem* __restrict__ items, const int32_t* __restrict__ bts,
    const int32_t* __restrict__ vbts, const int32_t* __restrict__ kbts,
    const AttnRow* __restrict__ arows,
    const float* __restrict__ rope_cos, const float* __restrict__ rope_sin,
    uint16_t* __restrict__ out, float* __restrict__ lse, float* __restrict__ split_o,
    float* __restrict__ split_lse, int n_q_heads, int n_kv_heads, int log2_page, float scale,
    float scale_log2e) {
  // double-buffered K and V^T tiles
  __shared__ __attribute__((aligned(16))) uint8_t kl[2][kKBytes];
  __shared__ __attribute__((aligned(16))) uint16_t vl[2][kVBytes / 2];
  // cos (dims 0 .. d/2-1) and sin (d/2 ..) at each row's position, per row
  // block: loaded once and shared by the block's four head waves (rows
  // padded by 4 floats so that the 32 rows of a fragment read fall in
  // different banks)
  // With K rotated on load the rotated queries move to LDS after the
  // prologue (8 KB per wave, over the cos/sin rows): the staging waves' K
  // rotation needs the 32 registers they would hold, which otherwise spill.
  constexpr int kRlBytes = R * kTileRows * (kD + 4) * 4;
  constexpr bool kQinLds = AK;
  constexpr int kQBytes = kQinLds ? 4 * R * 8 * 1024 : 0;
  __shared__ __attribute__((aligned(16))) uint8_t pro[kRlBytes > kQBytes ? kRlBytes : kQBytes];
  static_assert(4 * R * kOutLds <= (int)sizeof(pro), "outputs go through it");
  auto rl = reinterpret_cast<float (*)[kTileRows][kD + 4]>(pro);

  const AttnItem it = items[blockIdx.x];
  if (it.n_rows == 0) return;
  const int tid = threadIdx.x;
  const int wg = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = R == 1 ? wg : wg & 3;    // query head slot
  const int rb = R == 1 ? 0 : wg >> 2;   // row block
  const bool stager = R == 1 || wg < 4;  // waves that stage K and V
  const int lane = tid & 63;
  const int lrow = lane & 31;
  const int lh = lane >> 5;
  const int g = it.kv_head;
  const int page_mask = (1 << log2_page) - 1;
  // the K block table (pool pages flagged when K is rotated on load)
  const int32_t* bt = (AK ? kbts : bts) + it.bt_off;

  const int rbase = 32 * rb;
  // item rows are entries of arows: the computed row (q, out, lse) and
  // its position; items of consecutive computed rows at consecutive
  // positions carry their first row (crow0) and skip that read
  const int rr = min(rbase + lrow, it.n_rows - 1);
  int row, pos;
  if (it.crow0 >= 0) {
    row = it.crow0 + rr;
    pos = it.min_pos + rr;
  } else {
    const AttnRow ar = arows[it.row0 + rr];
    row = ar.row;
    pos = ar.pos;
  }
  const int pos_l = pos - 4 * lh;   // position less the lane's key offset in a tile
  // key tiles this wave's rows need: up to their largest position
  int my_ntiles = 0;
  if constexpr (R > 1) {
    int wmax = rbase + lrow < it.n_rows ? pos : -1;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wmax = max(wmax, __shfl_xor(wmax, o));
    my_ntiles = __builtin_amdgcn_readfirstlane(wmax + kKT) / kKT;
  }
  // wave w owns query head head0 + w of the group; with G < 4 the spare
  // waves recompute head G-1 and store nothing
  const int hl = G >= 4 ? it.head0 + w : min(w, G - 1);
  const bool wave_active = G >= 4 || w < G;

  bf16x8 qf[8];
  const uint8_t* qlds = pro + (tid >> 6) * 8192;
  auto qfrag = [&](int kst) __attribute__((always_inline)) -> bf16x8 {
    if constexpr (kQinLds) {
      Frag f;
      f.u = *reinterpret_cast<const uint4*>(qlds + kst * 1024 + lane * 16);
      return f.b;
    } else {
      return qf[kst];
    }
  };
  f32x16 o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[db][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;

  // ---- staging.  A tile's 32 keys form two 16-key blocks; with B >= 16
  // each block lies in one page.  Staging wave w takes block w / 2 and 64 of
  // its dims, so that a wave's page, and with it the base of its loads, is
  // uniform: scalar address arithmetic, one 32-bit offset a lane, and no
  // more than that held across a tile.
  // (With a wave over both blocks, per-lane bases and a range check on V the
  // kernel held 13 registers too many; RAG-8B 560 -> 532 us, its LOCAL form
  // 232 -> 216, Long-70B 8.97 -> 8.52 ms.)  A tile's raw V lives in vectors
  // local to one pass of the tile loop: as variables of the whole kernel it
  // was split into scalars and copied right after the loads, which waits for
  // them before the tile's products (10-15 % slower).
  // K: direct loads; lane l fetches key l % 16, 8-dim chunk l / 16 of 32
  //    dims, into its place in the fragment order (kKHalf).
  // V: lane l owns 16 bytes (dims 8 (l / 8) ..) of keys 2 (l % 8) and
  //    2 (l % 8) + 1, which sit next to each other in the permuted V^T row;
  //    each of its 8 dims takes one 4-byte write.
  const int sb = w >> 1;                   // 16-key block
  const uint32_t koff = ((lane & 15) * kD + 8 * (lane >> 4) + 64 * (w & 1)) * 2;
  const int kp = lane & 7;                 // key pair within the block
  const int vc8 = 64 * (w & 1) + 8 * (lane >> 3);   // first dim
  const uint32_t voff = (2 * kp * kD + vc8) * 2;
  const int vst = vc8 * kVStr + vt_col(16 * sb + 2 * kp);   // V^T element written
  // The pages of the wave's block of a tile (K, and V where it may differ):
  // uniform, so scalar loads, one tile before the tile's loads need them.
  auto fetch_pages = [&](int j, int& pk, int& pv) __attribute__((always_inline)) {
    const int i = min((j * kKT + 16 * sb) >> log2_page, it.n_pages - 1);
    pk = bt[i];
    if constexpr (AV || AK) pv = (AV ? vbts : bts)[it.bt_off + i];
  };
  auto block_base = [&](int page, int kq) -> int64_t {
    return ((((int64_t)page * n_kv_heads + g) << log2_page) + (kq & page_mask)) * kD;
  };
  auto load16 = [](const uint16_t* base, uint32_t off) __attribute__((always_inline)) {
    return *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint8_t*>(base) + off);
  };
  // Issues tile j's loads: K directly into the LDS buffer kt, V into
  // registers (written to LDS as V^T by store_tile).
  // K rotated on load: the lane's raw K of chunk kch of each RoPE half of
  // key kk, and whether the wave's block is a pool page
  const int kk = 16 * sb + (lane & 15), kch = (lane >> 4) + 4 * (w & 1);
  u32x4 kraw[2];
  bool krot = false;
  auto load_tile = [&](int j, int pk, int pv, uint8_t* kt, u32x4& v0, u32x4& v1)
      __attribute__((always_inline)) {
    const int key0 = j * kKT;
    const int kb0 = key0 + 16 * sb;
    const int64_t kbase = block_base(pk & ~kPoolPageFlag, kb0);
    const uint16_t* vsrc = vc;
    int64_t vbase = kbase;
    if constexpr (AV || AK) {
      if (AV && (pv & kPoolPageFlag)) vsrc = pool_v;
      vbase = block_base(pv & ~kPoolPageFlag, kb0);
    }
    uint32_t o0 = voff, o1 = voff + kD * 2;
    if (key0 + kKT > it.kv_len) {
      // Last, partial tile: keys past kv_len may be unwritten slots.  Their
      // scores are masked (a select), but 0 * NaN in P V would not be, so a
      // key of the tile stands in for them: the block's first, or the
      // tile's where the whole block lies past kv_len.  (Addresses are
      // replaced, not the loaded values: a select on those made tiles wait
      // for their loads here, before their products.)
      if (kb0 + 2 * kp >= it.kv_len) o0 = vc8 * 2;
      if (kb0 + 2 * kp + 1 >= it.kv_len) o1 = vc8 * 2;
      if (kb0 >= it.kv_len) {
        const int i = key0 >> log2_page;
        const int p0 = (AV ? vbts : bts)[it.bt_off + i];
        vsrc = (AV && (p0 & kPoolPageFlag)) ? pool_v : vc;
        vbase = block_base(p0 & ~kPoolPageFlag, key0);
      }
    }
    v0 = load16(vsrc + vbase, o0);
    v1 = load16(vsrc + vbase, o1);
    if constexpr (AK) {
      krot = (pk & kPoolPageFlag) != 0;
      if (krot) {   // through registers, rotated by store_k
        const uint16_t* src = pool_k + kbase;
        const uint32_t ko = ((lane & 15) * kD + 8 * kch) * 2;
        kraw[0] = load16(src, ko);
        kraw[1] = load16(src, ko + kD);
        return;
      }
    }
    const uint32_t kdst = lds_addr(kt) + sb * kKHalf + (w & 1) * 2 * kKBlk;
    lds_dma16<0>(kc + kbase, koff, kdst);
    lds_dma16<64>(kc + kbase, koff, kdst + kKBlk);
  };
  // K rotated on load: to LDS in fragment order
  auto store_k = [&](int j, uint8_t* kt) __attribute__((always_inline)) {
    float lo[8], hi[8], c[8], sn[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[2 * e] = bf16_to_f32(kraw[0][e] & 0xffffu);
      lo[2 * e + 1] = bf16_to_f32(kraw[0][e] >> 16);
      hi[2 * e] = bf16_to_f32(kraw[1][e] & 0xffffu);
      hi[2 * e + 1] = bf16_to_f32(kraw[1][e] >> 16);
    }
    const int pk = j * kKT + kk;
    load8(rope_cos + (int64_t)pk * (kD / 2) + 8 * kch, c);
    load8(rope_sin + (int64_t)pk * (kD / 2) + 8 * kch, sn);
    rope_rotate<8>(lo, hi, c, sn);
    uint4 a, b;
    a.x = f32_to_bf16(lo[0]) | (f32_to_bf16(lo[1]) << 16);
    a.y = f32_to_bf16(lo[2]) | (f32_to_bf16(lo[3]) << 16);
    a.z = f32_to_bf16(lo[4]) | (f32_to_bf16(lo[5]) << 16);
    a.w = f32_to_bf16(lo[6]) | (f32_to_bf16(lo[7]) << 16);
    b.x = f32_to_bf16(hi[0]) | (f32_to_bf16(hi[1]) << 16);
    b.y = f32_to_bf16(hi[2]) | (f32_to_bf16(hi[3]) << 16);
    b.z = f32_to_bf16(hi[4]) | (f32_to_bf16(hi[5]) << 16);
    b.w = f32_to_bf16(hi[6]) | (f32_to_bf16(hi[7]) << 16);
    uint8_t* dst = kt + sb * kKHalf + (kch >> 2) * kKBlk + (kch & 3) * 256 + (lane & 15) * 16;
    *reinterpret_cast<uint4*>(dst) = a;
    *reinterpret_cast<uint4*>(dst + 2 * kKBlk) = b;
  };
  auto store_tile = [&](const u32x4& v0, const u32x4& v1, uint16_t* vs)
      __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float f0 = e & 1 ? __uint_as_float(v0[e >> 1] & 0xffff0000u)
                             : __uint_as_float(v0[e >> 1] << 16);
      const float f1 = e & 1 ? __uint_as_float(v1[e >> 1] & 0xffff0000u)
                             : __uint_as_float(v1[e >> 1] << 16);
      *reinterpret_cast<uint32_t*>(vs + vst + e * kVStr) = pack_f16x2(f0, f1);
    }
  };
  // K fragment kst: the lane's key l % 32, dims 16 kst + 8 (l / 32) ..
  const int kfl = ((lane >> 4) & 1) * kKHalf + (lane >> 5) * 256 + (lane & 15) * 16;
  auto kfrag = [&](const uint8_t* ks, int kst) __attribute__((always_inline)) {
    return *reinterpret_cast<const uint4*>(ks + kfl + (kst >> 1) * kKBlk + (kst & 1) * 512);
  };

  // One 32-key tile: S^T = K Q^T, online softmax, O^T += V^T P^T.
  // MASK: kNoMask, kMaskCausal (keys past the row's position: tiles reaching
  // past the smallest row position of the item) or kMaskBoth (also keys
  // below kv_lo: the tile holding kv_lo).
  auto tile = [&](int j, auto mask_tag, const uint8_t* ks, const uint16_t* vs)
      __attribute__((always_inline)) {
    constexpr int MASK = decltype(mask_tag)::value;
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
    for (int kst = 0; kst < 8; ++kst) {
      Frag a;
      a.u = kfrag(ks, kst);
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.b, qfrag(kst), s, 0, 0, 0);
    }
    // keep four LDS fragment reads in flight ahead of the MFMAs
    // (scheduling groups: 0x100 = LDS read, 0x008 = MFMA)
    __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);

    // the V^T fragments of the first 16 keys are read while the softmax runs
    Frag va[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
      va[db].u = *reinterpret_cast<const uint4*>(vs + (32 * db + lrow) * kVStr + 8 * lh);
    if constexpr (MASK != kNoMask) {
      // score r holds key j kKT + 8 (r / 4) + 4 lh + r % 4: compare its
      // offset in the tile with the row's bounds moved to the same origin
      const int dhi = pos_l - j * kKT;
      const int dlo = it.kv_lo - 4 * lh - j * kKT;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int off = 8 * (r >> 2) + (r & 3);
        const bool out = MASK == kMaskBoth ? (off > dhi || off < dlo) : off > dhi;
        s[r] = out ? -INFINITY : s[r];
      }
    }
    // Online softmax with a lazily updated running max m, common to the
    // row's two half-waves.  P = exp2(s c - m c) is computed against the
    // current m and its per-lane sum checked: while the sum stays <= 2^kLazy
    // (so every P <= 2^kLazy, an exact range for fp16) no maximum is taken
    // and nothing is rescaled.  Otherwise (or while m is still -inf) the
    // tile's scores are computed again from the K tile in LDS, the maximum
    // moves m, O and l are rescaled, and P is recomputed.
    const float mc = m == -INFINITY ? 0.0f : m * scale_log2e;
    float ls[4];
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2e, -mc));
#pragma unroll
    for (int r = 0; r < 4; ++r) ls[r] = (s[r] + s[r + 4]) + (s[r + 8] + s[r + 12]);
    float lt = (ls[0] + ls[1]) + (ls[2] + ls[3]);
    // A row that sees no key up to here (in a key range of a split item past
    // its position) waits with m at -inf.
    const bool sees = MASK != kMaskCausal || pos_l >= j * kKT;
    if (__builtin_amdgcn_ballot_w64(!(lt <= kLazySum) || (m == -INFINITY && sees))) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
      for (int kst = 0; kst < 8; ++kst) {
        Frag a;
        a.u = kfrag(ks, kst);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.b, qfrag(kst), s, 0, 0, 0);
      }
      if constexpr (MASK != kNoMask) {
        const int dhi = pos_l - j * kKT;
        const int dlo = it.kv_lo - 4 * lh - j * kKT;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int off = 8 * (r >> 2) + (r & 3);
          const bool out = MASK == kMaskBoth ? (off > dhi || off < dlo) : off > dhi;
          s[r] = out ? -INFINITY : s[r];
        }
      }
      float mt = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mt = fmaxf(mt, s[r]);
      const float mn = fmaxf(m, fmaxf(mt, __shfl_xor(mt, 32)));
      const float alpha = mn == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f((m - mn) * scale_log2e);
      m = mn;
      l *= alpha;
#pragma unroll
      for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[db][r] *= alpha;
      const float mc2 = m == -INFINITY ? 0.0f : m * scale_log2e;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_exp2f(fmaf(s[r], scale_log2e, -mc2));
#pragma unroll
      for (int r = 0; r < 4; ++r) ls[r] = (s[r] + s[r + 4]) + (s[r + 8] + s[r + 12]);
    }
    f16x8 pf[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[h][e] = (_Float16)s[8 * h + e];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[db].h, pf[0], o[db], 0, 0, 0);
      va[db].u = *reinterpret_cast<const uint4*>(vs + (32 * db + lrow) * kVStr + 16 + 8 * lh);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      o[db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[db].h, pf[1], o[db], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    l += (ls[0] + ls[1]) + (ls[2] + ls[3]);
  };

  // keys kv_lo .. kv_len-1: tiles j0 .. ntiles-1.  A tile needs the mask
  // when it reaches past the smallest row position or starts below kv_lo.
  const int ntiles = (it.kv_len + kKT - 1) / kKT;
  const int j0 = it.kv_lo / kKT;
  const int jlo = min(ntiles, (it.kv_lo + kKT - 1) / kKT);   // first tile without keys < kv_lo
  const int nfull = min(ntiles, (it.min_pos + 1) / kKT);      // tiles ending at or before min_pos
  // page ids of the next tile to load (staging waves; the first tile's
  // come with the item)
  int pp0 = sb ? it.pg[1] : it.pg[0], pp1 = 0;
  if (AV || AK) fetch_pages(j0, pp0, pp1);
  // One tile j: issue the next tile's loads into the other buffers, compute
  // this one, stage the next V^T, wait for this wave's direct K loads, then
  // the workgroup barrier.
  // SKIP: tiles past a row block's last row occur only in the masked tail.
  auto run_tiles = [&](int ja, int jb, auto mask_tag, auto skip_tag)
      __attribute__((always_inline)) {
    constexpr bool SKIP = R > 1 && decltype(skip_tag)::value;
    for (int j = ja; j < jb; ++j) {
      const bool more = j + 1 < ntiles;
      u32x4 v0, v1;
      if (more) {
        load_tile(j + 1, pp0, pp1, kl[(j + 1) & 1], v0, v1);
        fetch_pages(j + 2, pp0, pp1);
      }
      if (!SKIP || j < my_ntiles) tile(j, mask_tag, kl[j & 1], vl[j & 1]);
      if (more) {
        store_tile(v0, v1, vl[(j + 1) & 1]);
        if (AK && krot) store_k(j + 1, kl[(j + 1) & 1]);
      }
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __syncthreads();
    }
  };
  // The waves of the other row blocks stage nothing and skip the tiles past
  // their own rows (fully masked for them; all tiles for a row block past
  // the item's last row).  Kept as a separate loop: with the staging under
  // a wave-dependent condition in one loop the compiler kept the staging
  // registers live in every wave and spilled.
  auto run_tiles_ns = [&](int ja, int jb, auto mask_tag) __attribute__((always_inline)) {
    for (int j = ja; j < jb; ++j) {
      if (j < my_ntiles) tile(j, mask_tag, kl[j & 1], vl[j & 1]);
      __syncthreads();
    }
  };
  u32x4 vf0, vf1;
  if (stager) {
    load_tile(j0, pp0, pp1, kl[j0 & 1], vf0, vf1);
    fetch_pages(j0 + 1, pp0, pp1);
  }
  // While the first tile is in flight: each row block's cos/sin rows go to
  // LDS (thread t of the block loads 8 dims of cos and sin of row t / 8)
  // and every wave loads its raw queries; the rotation follows the barrier.
  {
    const int t = tid & 255, lr = t >> 3, c8 = 8 * (t & 7);
    const int pr = min(rbase + lr, it.n_rows - 1);
    const int ppos = it.crow0 >= 0 ? it.min_pos + pr : arows[it.row0 + pr].pos;
    float c[8], sn[8];
    load8(rope_cos + (int64_t)ppos * (kD / 2) + c8, c);
    load8(rope_sin + (int64_t)ppos * (kD / 2) + c8, sn);
    store8(&rl[rb][lr][c8], c);
    store8(&rl[rb][lr][kD / 2 + c8], sn);
  }
  uint4 qraw[8];
  {
    const uint16_t* qp = q + ((int64_t)row * n_q_heads + g * G + hl) * kD;
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int d0 = 16 * ks + 8 * lh;
      qraw[ks] = *reinterpret_cast<const uint4*>(qp + d0);
      qraw[ks + 4] = *reinterpret_cast<const uint4*>(qp + d0 + kD / 2);
    }
  }
  if (stager) {
    store_tile(vf0, vf1, vl[j0 & 1]);
    if (AK && krot) store_k(j0, kl[j0 & 1]);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  __syncthreads();
  // ---- rotated queries as bf16 B operands: lane = query row, k = head dim
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int d0 = 16 * ks + 8 * lh;
    float lo[8], hi[8], c[8], sn[8];
    const uint32_t wl[4] = {qraw[ks].x, qraw[ks].y, qraw[ks].z, qraw[ks].w};
    const uint32_t wh[4] = {qraw[ks + 4].x, qraw[ks + 4].y, qraw[ks + 4].z, qraw[ks + 4].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      lo[2 * e] = bf16_to_f32(wl[e] & 0xffffu);
      lo[2 * e + 1] = bf16_to_f32(wl[e] >> 16);
      hi[2 * e] = bf16_to_f32(wh[e] & 0xffffu);
      hi[2 * e + 1] = bf16_to_f32(wh[e] >> 16);
    }
    load8(&rl[rb][lrow][d0], c);
    load8(&rl[rb][lrow][kD / 2 + d0], sn);
    rope_rotate<8>(lo, hi, c, sn);
    Frag a, b;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      a.w[e] = pack_bf16x2(lo[2 * e], lo[2 * e + 1]);
      b.w[e] = pack_bf16x2(hi[2 * e], hi[2 * e + 1]);
    }
    qf[ks] = a.b;
    qf[ks + 4] = b.b;
  }
  if constexpr (kQinLds) {
    __syncthreads();   // every wave has read its cos/sin rows
#pragma unroll
    for (int kst = 0; kst < 8; ++kst) {
      Frag f;
      f.b = qf[kst];
      *reinterpret_cast<uint4*>(pro + (tid >> 6) * 8192 + kst * 1024 + lane * 16) = f.u;
    }
  }
  if (stager) {
    run_tiles(j0, jlo, MaskBoth{}, std::false_type{});
    run_tiles(jlo, max(jlo, nfull), NoMask{}, std::false_type{});
    run_tiles(max(jlo, nfull), ntiles, MaskCausal{}, std::true_type{});
  } else {
    run_tiles_ns(j0, jlo, MaskBoth{});
    run_tiles_ns(jlo, max(jlo, nfull), NoMask{});
    run_tiles_ns(max(jlo, nfull), ntiles, MaskCausal{});
  }

  // ---- epilogue: normalise, round to bf16, store rows of this tile
  const float lt = l + __shfl_xor(l, 32);
  const int n_mine = min(kTileRows, it.n_rows - rbase);   // this row block's rows
  if (!wave_active || n_mine <= 0) return;
  float inv = 1.0f / lt;
  if (it.part_slot >= 0) {
    // one key range of a split item: normalized rows and log-sum-exp in
    // fp32 to this row block's slot, merged by attn_merge_kernel; a row
    // that sees no key of the range weighs nothing there (0, -inf).  (A row
    // whose scores in it are all NaN has no maximum either, but its sum is
    // NaN.)
    if (lrow >= n_mine) return;
    const bool none = m == -INFINITY && lt == 0.0f;
    if (none) inv = 0.0f;
    const int64_t slot = it.part_slot + (int64_t)rb * it.n_parts;
    const int64_t sr = (slot * kTileRows + lrow) * kSplitHeads + w;
    float* po = split_o + sr * kD;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int rg = 0; rg < 4; ++rg)
        *reinterpret_cast<float4*>(po + 32 * db + 8 * rg + 4 * lh) =
            make_float4(o[db][4 * rg] * inv, o[db][4 * rg + 1] * inv,
                        o[db][4 * rg + 2] * inv, o[db][4 * rg + 3] * inv);
    if (lh == 0) split_lse[sr] = none ? -INFINITY : m * scale + logf(lt);
    return;
  }
  const int hq = g * G + (G >= 4 ? it.head0 : 0) + w;
  if (lse && lh == 0 && lrow < n_mine)
    lse[(int64_t)row * n_q_heads + hq] = m * scale + logf(lt);
  // (the cos/sin rows' LDS is free: every wave is past the last tile's barrier)
  store_out(o, inv, pro + (tid >> 6) * kOutLds, lane, n_mine, out, [&](int r) -> int64_t {
    const int cr = it.crow0 >= 0 ? it.crow0 + rbase + r : arows[it.row0 + rbase + r].row;
    return ((int64_t)cr * n_q_heads + hq) * kD;
  });
}

int ilog2(int x) {
  int l = 0;
  while ((1 << l) < x) ++l;
  return l;
}

// Merge of a split item's key ranges (Section 5.3's extend pass over the
// whole prompt, run as several ranges): for its row r and query head
// hq0 + hs, from the ranges' normalized outputs o_c and log-sum-exps lse_c,
//   lse = log sum_c exp(lse_c),   o = sum_c exp(lse_c - lse) o_c,
// o rounded to bf16 once.
//
// Bound by latency: the partial rows have just been left in the caches, and
// a launch merges a few thousand of them.  Half a wave takes one (row, head):
// its 32 lanes read the 512 bytes of a partial row together and lane c % 32
// holds the weight of range c.  The first kMergeAhead rows and the log-sum-exps
// are all asked for at once, so a pair costs the merge descriptor's latency
// and one more.  kMergeCut workgroups share a row block of a split item.
// (Before: two pairs a half-wave in turn, each waiting for its log-sum-exps
// before its rows.  A layer of one RAG request with every chunk cached 53.2 ->
// 48.8 us, of which the merge had 9.)
constexpr int kMergeCut = 16;
constexpr int kMergePairs = kTileRows * kSplitHeads / kMergeCut;   // (row, head)s each
constexpr int kMergeAhead = 8;
static_assert(kMergePairs == 8, "one a half-wave");

__global__ __launch_bounds__(256) void attn_merge_kernel(
    const CombineDesc* __restrict__ cds, const AttnRow* __restrict__ arows,
    const float* __restrict__ split_o, const float* __restrict__ split_lse,
    uint16_t* __restrict__ out, float* __restrict__ lse, int n_q_heads) {
  const CombineDesc cd = cds[blockIdx.x];
  const int lane = threadIdx.x & 31;
  const int pair = blockIdx.y * kMergePairs + (threadIdx.x >> 5);
  const int r = pair / kSplitHeads, hs = pair % kSplitHeads;
  if (r >= cd.n_rows || hs >= cd.n_heads) return;
  auto slot_row = [&](int c) -> int64_t {
    return ((int64_t)(cd.slot0 + c) * kTileRows + r) * kSplitHeads + hs;
  };
  auto part = [&](int c) {
    return *reinterpret_cast<const float4*>(split_o + slot_row(c) * kD + 4 * lane);
  };
  auto range_lse = [&](int c) { return c < cd.n_slots ? split_lse[slot_row(c)] : -INFINITY; };
  const float l0 = range_lse(lane);
  const int row = arows[cd.row0 + r].row;
  float4 ahead[kMergeAhead];   // past the last range: its row again, unused
#pragma unroll
  for (int c = 0; c < kMergeAhead; ++c) ahead[c] = part(min(c, cd.n_slots - 1));
  float mx = l0;
  for (int c = lane + 32; c < cd.n_slots; c += 32) mx = fmaxf(mx, range_lse(c));
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
  float den = expf(l0 - mx);
  for (int c = lane + 32; c < cd.n_slots; c += 32) den += expf(range_lse(c) - mx);
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) den += __shfl_xor(den, o);
  const float ltot = mx + logf(den);
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  auto add = [&](float wc, const float4& v) {
    acc.x = fmaf(wc, v.x, acc.x);
    acc.y = fmaf(wc, v.y, acc.y);
    acc.z = fmaf(wc, v.z, acc.z);
    acc.w = fmaf(wc, v.w, acc.w);
  };
  float wl = expf(l0 - ltot);
#pragma unroll
  for (int c = 0; c < kMergeAhead; ++c) {
    const float wc = __shfl(wl, c, 32);
    if (c < cd.n_slots) add(wc, ahead[c]);
  }
  for (int c = kMergeAhead; c < cd.n_slots; ++c) {
    if (c % 32 == 0) wl = expf(range_lse(c + lane) - ltot);
    add(__shfl(wl, c % 32, 32), part(c));
  }
  const int64_t orow = (int64_t)row * n_q_heads + cd.hq0 + hs;
  uint2 v;
  v.x = f32_to_bf16(acc.x) | (f32_to_bf16(acc.y) << 16);
  v.y = f32_to_bf16(acc.z) | (f32_to_bf16(acc.w) << 16);
  *reinterpret_cast<uint2*>(out + orow * kD + 4 * lane) = v;
  if (lse && lane == 0) lse[orow] = ltot;
}

}  // namespace

hipError_t launch_attn(const tsr_plan* p, int32_t part, const AttnItem* items,
                       int32_t n_items, const void* pool_k, const void* pool_v,
                       const void* q, const void* req_k, const void* req_v, void* out,
                       float* lse, hipStream_t s) {
  if (n_items == 0 || p->T == 0) return hipSuccess;
  const tsr_model& m = p->model;
  const int lp = ilog2(m.page_size);
  const int G = m.n_q_heads / m.n_kv_heads;
  const dim3 grid(n_items);
  if (m.act_dtype == TSR_F32) {
#define TSR_F32K(DIM)                                                             \
  hipLaunchKernelGGL(attn_f32_kernel<DIM>, dim3(n_items, G, kTileRows / kF32Rows), \
                     dim3(64 * kF32Waves<DIM>), 0, s,                             \
                     static_cast<const float*>(q), static_cast<const float*>(req_k), \
                     static_cast<const float*>(req_v), items,                       \
                     p->dev.block_tables, p->dev.rows, p->dev.rope_cos,            \
                     p->dev.rope_sin, static_cast<float*>(out), lse, m.n_q_heads,  \
                     m.n_kv_heads, lp, p->scale)
    switch (m.head_dim) {
      case 64: TSR_F32K(64); break;
      case 128: TSR_F32K(128); break;
      case 256: TSR_F32K(256); break;
      default: return hipErrorInvalidValue;
    }
#undef TSR_F32K
    return hipGetLastError();
  }
  if (p->row_blocks == kPipeRowBlocks)
    return launch_attn_pipe(p, items, n_items, pool_v, q, req_k, req_v, out, lse, s);
  const float sl2e = (float)((double)p->scale * 1.4426950408889634);
#define TSR_MFMA(GG, AV, AK)                                                       \
  if (p->row_blocks == kMaxRowBlocks)                                              \
    TSR_MFMA_R(GG, AV, AK, kMaxRowBlocks);                                         \
  else                                                                             \
    TSR_MFMA_R(GG, AV, AK, 1)
#define TSR_MFMA_R(GG, AV, AK, RB)                                                 \
  hipLaunchKernelGGL((attn_mfma_kernel<GG, AV, AK, RB>), grid, dim3(256 * (RB)), 0, s, \
                     static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(req_k), \
                     static_cast<const uint16_t*>(req_v),                          \
                     static_cast<const uint16_t*>(pool_k),                         \
                     static_cast<const uint16_t*>(pool_v), items,                  \
                     p->dev.block_tables, p->dev.v_block_tables,                    \
                     p->dev.k_block_tables, p->dev.attn_rows, p->dev.rope_cos,      \
                     p->dev.rope_sin, static_cast<uint16_t*>(out), lse,             \
                     p->dev.split_o, p->dev.split_lse, m.n_q_heads, m.n_kv_heads, lp, \
                     p->scale, sl2e)
#define TSR_MFMA_G(GG)                                                             \
  if (p->alias_v && p->alias_k) TSR_MFMA(GG, true, true);                          \
  else if (p->alias_v) TSR_MFMA(GG, true, false);                                  \
  else if (p->alias_k) TSR_MFMA(GG, false, true);                                  \
  else TSR_MFMA(GG, false, false)
  switch (G) {
    case 1: TSR_MFMA_G(1); break;
    case 2: TSR_MFMA_G(2); break;
    case 4: TSR_MFMA_G(4); break;
    case 8: TSR_MFMA_G(8); break;
    default: return hipErrorInvalidValue;
  }
#undef TSR_MFMA_G
#undef TSR_MFMA
#undef TSR_MFMA_R
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p->n_combine == 0) return e;
  // the split items of this part: part 0's merge descriptors come first
  const int32_t c0 = part == TSR_ATTN_AFTER_COMPOSE ? p->n_combine_part[0] : 0;
  const int32_t nc = part == TSR_ATTN_ALL ? p->n_combine : p->n_combine_part[part - 1];
  if (nc == 0) return hipSuccess;
  hipLaunchKernelGGL(attn_merge_kernel, dim3(nc, kMergeCut), dim3(256), 0, s,
                     p->dev.combine + c0,
                     p->dev.attn_rows, p->dev.split_o, p->dev.split_lse, static_cast<uint16_t*>(out), lse,
                     m.n_q_heads);
  return hipGetLastError();
}

}  // namespace tsr
