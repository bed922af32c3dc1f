// Causal GQA prefill attention over an e4m3 request KV (codes + one
// power-of-two scale per (page, K|V)).  Same work decomposition, 32-key tile
// schedule and online softmax as the bf16 kernel (attn.hip); what differs:
//
//   * rotated queries are quantized to e4m3 per (row, head) with the
//     smallest power-of-two scale covering the row (a kernel choice that the
//     CPU oracle mirrors exactly);
//   * S^T = K Q^T runs on the codes with v_mfma_scale_f32_32x32x64_f8f6f4
//     (unit block scales); the row's Q scale and each key's page scale are
//     applied to S afterwards (per lane: one row, four pages per tile);
//   * V codes are dequantized to fp16 (exact for e4m3 values times a
//     power-of-two scale up to 2^7, the most that keeps every code inside
//     fp16's range; a page with a larger V scale becomes NaN, so outputs
//     that depend on it are non-finite rather than silently clipped) while
//     being transposed into LDS,
//     and P V runs in fp16 MFMA as in the bf16 kernel, so P keeps fp16
//     precision (e4m3 P would cost several percent of relative error).
#include <cmath>
#include <type_traits>

#include "attn_common.h"
#include "kernels_common.h"
#include "tsr_internal.h"

namespace tsr {

namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// An e4m3 K tile in LDS: for each 16-key block and 64-dim step kst a 1 KB
// block in which 16-byte chunk c of key k lies at 256 c + 16 k.  One direct
// load by a wave that reads one page fills a 1 KB block, and a fragment (32
// bytes of a key) is two 16-byte reads in 256-byte runs.
constexpr int kK8Blk = 1024;
constexpr int kK8Bytes = 4 * kK8Blk;
constexpr int kVElems = kD * kVStr;

__device__ __forceinline__ int page_scale_exp(float amax) {
  if (!(amax > 0.0f)) return 0;
  int e;
  const float mfr = frexpf(amax, &e);
  return mfr <= 0.875f ? e - 9 : e - 8;
}

// R: row blocks per workgroup.  Waves 4 b .. 4 b + 3 own the 32 rows of
// row block b; the first four waves stage every K/V tile for all of them
// (three row blocks share each staged tile, which cuts the KV reads per row
// threefold).
// KS: wave groups per row block (R = 1).  The item's key tiles are dealt to
// KS groups of four waves, each staging its own tiles and keeping its own
// running softmax; group 0 merges them through LDS at the end.  Used where a
// launch has too few items to fill the chip: it then lasts as long as its
// longest item, and the groups cut that into KS parts.
template <int G, int R, int KS>
__global__ __launch_bounds__(256 * R * KS, 3) void attn_fp8_kernel(
    const uint16_t* __restrict__ q, const uint8_t* __restrict__ kc,
    const uint8_t* __restrict__ vc, const float* __restrict__ scales,
    const AttnItem* __restrict__ items, const int32_t* __restrict__ bts,
    const AttnRow* __restrict__ arows, const float* __restrict__ rope_cos,
    const float* __restrict__ rope_sin, uint16_t* __restrict__ out,
    float* __restrict__ lse, int n_q_heads, int n_kv_heads, int log2_page,
    float scale_log2e) {
  constexpr int HPW = 1;  // query heads per wave
  static_assert(KS == 1 || (KS == 3 && R == 1), "wave groups");
  __shared__ __attribute__((aligned(16))) uint8_t klds[KS][2][kK8Bytes];
  __shared__ __attribute__((aligned(16))) uint16_t vlds[KS][2][kVElems];
  // K page scales of each staged tile's two 16-key blocks
  __shared__ float slds[KS][2][2];
  // cos (dims 0 .. d/2-1) and sin (d/2 ..) at each row's position, per row
  // block, loaded once and shared by its four head waves (rows padded by 4
  // floats so that the 32 rows of a fragment read fall in different banks)
  __shared__ __attribute__((aligned(16))) float rl[R][32][kD + 4];

  const AttnItem it = items[blockIdx.x];
  if (it.n_rows == 0) return;
  const int tid = threadIdx.x;
  const int wg = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = wg & 3;                  // query head slot
  const int rb = KS == 1 ? wg >> 2 : 0;  // row block
  const int kg = KS == 1 ? 0 : wg >> 2;  // wave group
  const bool stager = KS > 1 || wg < 4;  // waves that stage K and V
  auto kmem = klds[kg];
  auto vmem = vlds[kg];
  auto kscl = slds[kg];
  const int lane = tid & 63;
  const int lrow = lane & 31;
  const int lh = lane >> 5;
  const int g = it.kv_head;
  const int page_mask = (1 << log2_page) - 1;
  const int32_t* bt = bts + it.bt_off;
  const int rbase = 32 * rb;
  // item rows are entries of arows: the computed row (q, out, lse) and
  // its position (with three row blocks, each request's rows grouped by
  // first visible key); items of consecutive computed rows at consecutive
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
  // ---- staging.  The two 16-key blocks of a tile each lie in one page;
  // staging wave w takes block w / 2 and 64 of its dims, so that a wave's
  // page, the base of its loads and its page scales are uniform.
  // K: one direct load a wave; lane l fetches 16 bytes (chunk l / 16 of the
  //    64) of key l % 16 into their place in the fragment order.
  // V: lane l owns 8 bytes (dims 8 (l / 8) ..) of keys 2 (l % 8) and
  //    2 (l % 8) + 1, which sit next to each other in the permuted V^T row.
  // Page ids are fetched a tile before the loads that need them, and raw V
  // is local to one pass of the tile loop (carried around it, it is copied
  // right after the loads, which waits for them there).
  // (Before: K through registers, both blocks a wave, page ids loaded with the
  // tile and the first tile after the queries.  fp8 RAG 1,712 -> 1,640 us,
  // one fp8 request 225 -> 203.)
  const int sb = w >> 1;
  const uint32_t koff = (lane & 15) * kD + 16 * (lane >> 4) + 64 * (w & 1);
  const int kp = lane & 7;
  const int vc8 = 64 * (w & 1) + 8 * (lane >> 3);
  const uint32_t voff = 2 * kp * kD + vc8;
  const int vst = vc8 * kVStr + vt_col(16 * sb + 2 * kp);
  auto fetch_page = [&](int j) __attribute__((always_inline)) {
    return bt[min((j * kKT + 16 * sb) >> log2_page, it.n_pages - 1)];
  };
  auto block_base = [&](int page, int kq) -> int64_t {
    return ((((int64_t)page * n_kv_heads + g) << log2_page) + (kq & page_mask)) * kD;
  };
  auto load_tile = [&](int j, int page, uint8_t* kt, u32x2& v0, u32x2& v1, float& nk, float& nv)
      __attribute__((always_inline)) {
    const int key0 = j * kKT;
    const int kb0 = key0 + 16 * sb;
    const int64_t base = block_base(page, kb0);
    nk = scales[2 * (int64_t)page];
    nv = scales[2 * (int64_t)page + 1];
    const uint8_t* vsrc = vc + base;
    uint32_t o0 = voff, o1 = voff + kD;
    if (key0 + kKT > it.kv_len) {
      // last, partial tile: keys past kv_len may be unwritten slots.  Their
      // scores are masked (a select), but 0 * NaN in P V would not be, so a
      // key of the tile stands in for them: the block's first, or the
      // tile's where the whole block lies past kv_len
      if (kb0 + 2 * kp >= it.kv_len) o0 = vc8;
      if (kb0 + 2 * kp + 1 >= it.kv_len) o1 = vc8;
      if (kb0 >= it.kv_len) {
        const int p0 = bt[key0 >> log2_page];
        vsrc = vc + block_base(p0, key0);
        nv = scales[2 * (int64_t)p0 + 1];
      }
    }
    v0 = *reinterpret_cast<const u32x2*>(vsrc + o0);
    v1 = *reinterpret_cast<const u32x2*>(vsrc + o1);
    lds_dma16<0>(kc + base, koff, lds_addr(kt) + (2 * sb + (w & 1)) * kK8Blk);
  };
  auto store_tile = [&](int buf, const u32x2& v0, const u32x2& v1, float nk, float nv)
      __attribute__((always_inline)) {
    if ((w & 1) == 0 && lane == 0) kscl[buf][sb] = nk;
    // V^T[d][key] in fp16: gather byte e of keys (k0, k1) into one word and
    // convert two codes at a time with the page scale.
    // a page scale above 2^7 can take codes (|c| <= 448) past fp16's
    // 65504: such pages are refused loudly, as NaN values
    const float s = nv <= 128.0f ? nv : __builtin_nanf("");
    uint16_t* vs = vmem[buf] + vst;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int e2 = 0; e2 < 2; ++e2) {
        // bytes (k0[e], k1[e], k0[e+1], k1[e+1]) for e = 2*e2 within the word
        const uint32_t sel = e2 ? 0x07030602u : 0x05010400u;
        const uint32_t p01 = __builtin_amdgcn_perm(v1[half], v0[half], sel);
        // low word: keys (0,1) at dim e; high word: at dim e + 1
        const f16x2 l01 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(p01, s, false);
        const f16x2 h01 = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(p01, s, true);
        const int d = 4 * half + 2 * e2;
        *reinterpret_cast<uint32_t*>(vs + d * kVStr) = __builtin_bit_cast(uint32_t, l01);
        *reinterpret_cast<uint32_t*>(vs + (d + 1) * kVStr) = __builtin_bit_cast(uint32_t, h01);
      }
    }
  };
  // keys kv_lo .. kv_len-1: tiles j0 .. ntiles-1; a tile needs the mask when
  // it reaches past the smallest row position or starts below kv_lo
  const int ntiles = (it.kv_len + kKT - 1) / kKT;
  const int j0 = it.kv_lo / kKT;
  const int jlo = (it.kv_lo + kKT - 1) / kKT;
  const int nfull = min(ntiles, (it.min_pos + 1) / kKT);
  // the first tile's loads (its page comes with the item) run under the
  // query rotation
  int npage = sb ? it.pg[1] : it.pg[0];
  int j = j0 + kg;   // this wave group's tile
  if (KS > 1 && kg > 0) npage = fetch_page(j);
  u32x2 vf0, vf1;
  float nkf = 1.0f, nvf = 1.0f;
  const bool first = stager && (KS == 1 || j < ntiles);
  if (first) {
    load_tile(j, npage, kmem[j & 1], vf0, vf1, nkf, nvf);
    npage = fetch_page(j + KS);
  }
  if (KS == 1 || kg == 0) {
    const int t = tid & 255, lr = t >> 3, c8 = 8 * (t & 7);
    const int pr = min(rbase + lr, it.n_rows - 1);
    const int ppos = it.crow0 >= 0 ? it.min_pos + pr : arows[it.row0 + pr].pos;
    float c[8], sn[8];
    load8(rope_cos + (int64_t)ppos * (kD / 2) + c8, c);
    load8(rope_sin + (int64_t)ppos * (kD / 2) + c8, sn);
    store8(&rl[rb][lr][c8], c);
    store8(&rl[rb][lr][kD / 2 + c8], sn);
  }
  // key tiles this wave's rows need: up to their largest position
  int my_ntiles = 1 << 30;
  if constexpr (R > 1) {
    int wmax = rbase + lrow < it.n_rows ? pos : -1;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wmax = max(wmax, __shfl_xor(wmax, o));
    my_ntiles = __builtin_amdgcn_readfirstlane(wmax + kKT) / kKT;
  }
  // ---- queries: rotate in fp32, quantize per (row, head) to e4m3.  Lane
  // half lh holds dims [32 lh, 32 lh + 32) of both RoPE halves, i.e. the
  // B operands of the two 64-deep k steps.  The raw rows are on their way
  // while the cos/sin rows go to LDS.
  i32x8 qf[HPW][2];
  float qs[HPW];
  uint4 qraw[HPW][8];
#pragma unroll
  for (int i = 0; i < HPW; ++i) {
    // wave w owns query head head0 + w of the group; with G < 4 the spare
    // waves recompute head G-1 and store nothing
    const int hl = G >= 4 ? it.head0 + w + 4 * i : min(w + 4 * i, G - 1);
    const uint16_t* qp = q + ((int64_t)row * n_q_heads + g * G + hl) * kD + 32 * lh;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      qraw[i][c] = *reinterpret_cast<const uint4*>(qp + 8 * c);
      qraw[i][c + 4] = *reinterpret_cast<const uint4*>(qp + 8 * c + kD / 2);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < HPW; ++i) {
    float lo[32], hi[32];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int d0 = 32 * lh + 8 * c;
      const uint4 a = qraw[i][c], b = qraw[i][c + 4];
      const uint32_t wl[4] = {a.x, a.y, a.z, a.w}, wh[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo[8 * c + 2 * e] = bf16_to_f32(wl[e] & 0xffffu);
        lo[8 * c + 2 * e + 1] = bf16_to_f32(wl[e] >> 16);
        hi[8 * c + 2 * e] = bf16_to_f32(wh[e] & 0xffffu);
        hi[8 * c + 2 * e + 1] = bf16_to_f32(wh[e] >> 16);
      }
      float cs[8], sn[8];
      load8(&rl[rb][lrow][d0], cs);
      load8(&rl[rb][lrow][kD / 2 + d0], sn);
      rope_rotate<8>(lo + 8 * c, hi + 8 * c, cs, sn);
    }
    float amax = 0.0f;
#pragma unroll
    for (int e = 0; e < 32; ++e) amax = fmaxf(amax, fmaxf(fabsf(lo[e]), fabsf(hi[e])));
    amax = fmaxf(amax, __shfl_xor(amax, 32));
    const int ek = page_scale_exp(amax);
    qs[i] = ldexpf(1.0f, ek);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const float* x = half ? hi : lo;
#pragma unroll
      for (int wd = 0; wd < 8; ++wd) {
        float a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          a[e] = fminf(fmaxf(ldexpf(x[4 * wd + e], -ek), -448.0f), 448.0f);
        int p = __builtin_amdgcn_cvt_pk_fp8_f32(a[0], a[1], 0, false);
        p = __builtin_amdgcn_cvt_pk_fp8_f32(a[2], a[3], p, true);
        qf[i][half][wd] = p;
      }
    }
  }

  f32x16 o[HPW][4];
  float m[HPW], l[HPW];
#pragma unroll
  for (int i = 0; i < HPW; ++i) {
    m[i] = -INFINITY;
    l[i] = 0.0f;
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[i][db][r] = 0.0f;
  }
  bool wave_active[HPW];
#pragma unroll
  for (int i = 0; i < HPW; ++i) wave_active[i] = G >= 4 || (w + 4 * i) < G;

  // K fragment kst: the lane's key l % 32, dims 64 kst + 32 (l / 32) ..; both
  // 16-byte halves land in adjacent registers of the operand
  const int kfl = (lrow >> 4) * 2 * kK8Blk + 512 * lh + 16 * (lrow & 15);
  auto kfrag = [&](const uint8_t* ks, int kst) __attribute__((always_inline)) {
    union { uint4 u[2]; i32x8 v; } x;
    x.u[0] = *reinterpret_cast<const uint4*>(ks + kfl + kst * kK8Blk);
    x.u[1] = *reinterpret_cast<const uint4*>(ks + kfl + kst * kK8Blk + 256);
    return x.v;
  };
  // MASK: 0 none, 1 keys past the row's position (tiles reaching past the
  // item's smallest position), 2 also keys below kv_lo (the tile holding it)
  auto tile = [&](int j, auto mask_tag) {
    constexpr int MASK = decltype(mask_tag)::value;
    const uint8_t* ks = kmem[j & 1];
    const uint16_t* vs = vmem[j & 1];
    f32x16 s[HPW][1];
#pragma unroll
    for (int i = 0; i < HPW; ++i)
#pragma unroll
      for (int kb = 0; kb < 1; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[i][kb][r] = 0.0f;
#pragma unroll
    for (int kst = 0; kst < 2; ++kst) {
#pragma unroll
      for (int kb = 0; kb < 1; ++kb) {
        const i32x8 a = kfrag(ks, kst);
#pragma unroll
        for (int i = 0; i < HPW; ++i)
          s[i][kb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
              a, qf[i][kst], s[i][kb], 0, 0, 0, 127, 0, 127);
      }
    }
    // the V^T fragments of the first 16 keys are read while the softmax runs
    Frag va[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
      va[db].u = *reinterpret_cast<const uint4*>(vs + (32 * db + lrow) * kVStr + 8 * lh);
    // page of S register r: r/8 within the tile; its factor f (Q scale x K
    // page scale x softmax scale x log2 e) is > 0, so P = exp2(f s - m) is
    // one fma and one exp2 per score and each page's row max is f times the
    // max of its raw scores.
    // Lazy rescale on the tile's probability sum (as in attn.hip): P is
    // taken against the running max m; while a lane's sum stays <= 2^kLazy
    // (every P is then exact-range for fp16) no max is taken.  Otherwise
    // (or while m is still -inf) the scores are computed again from the
    // tile in LDS, m moves to the row max, O and l are rescaled and P is
    // recomputed.
    auto scores = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[i][0][r] = 0.0f;
#pragma unroll
      for (int kst = 0; kst < 2; ++kst) {
        s[i][0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
            kfrag(ks, kst), qf[i][kst], s[i][0], 0, 0, 0, 127, 0, 127);
      }
    };
    auto mask = [&](int i) __attribute__((always_inline)) {
      if constexpr (MASK != 0) {
        // score r holds key j kKT + 8 (r / 4) + 4 lh + r % 4: compare its
        // in-tile offset with the row's bounds moved to the same origin
        const int dhi = pos - 4 * lh - j * kKT;
        const int dlo = it.kv_lo - 4 * lh - j * kKT;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int off = 8 * (r >> 2) + (r & 3);
          const bool out = MASK == 2 ? (off > dhi || off < dlo) : off > dhi;
          s[i][0][r] = out ? -INFINITY : s[i][0][r];
        }
      }
    };
    f16x8 pf[HPW][2];
#pragma unroll
    for (int i = 0; i < HPW; ++i) {
      float f[2];
#pragma unroll
      for (int b = 0; b < 2; ++b) f[b] = qs[i] * kscl[j & 1][b] * scale_log2e;
      mask(i);
      // row sum in fp32 as four independent chains of plain adds; a row with
      // no visible key yet keeps m at -inf and is exponentiated against 0
      const float mi = m[i] == -INFINITY ? 0.0f : m[i];
      float ls[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(s[i][0][r], f[r >> 3], -mi));
        s[i][0][r] = p;
        ls[r & 3] += p;
      }
      const float lt = (ls[0] + ls[1]) + (ls[2] + ls[3]);
      // a row that sees no key of its wave group's tiles up to here waits
      // with m at -inf
      const bool sees = KS == 1 || MASK != 1 || pos - 4 * lh >= j * kKT;
      if (__builtin_amdgcn_ballot_w64(!(lt <= kLazySum) || (m[i] == -INFINITY && sees))) {
        scores(i);
        mask(i);
        float mb[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          float x = s[i][0][8 * b];
#pragma unroll
          for (int r = 1; r < 8; ++r) x = fmaxf(x, s[i][0][8 * b + r]);
          mb[b] = x * f[b];
        }
        const float mt = fmaxf(mb[0], mb[1]);
        const float mn = fmaxf(m[i], fmaxf(mt, __shfl_xor(mt, 32)));
        const float alpha = mn == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m[i] - mn);
        m[i] = mn;
        l[i] *= alpha;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[i][db][r] *= alpha;
        const float mi2 = m[i] == -INFINITY ? 0.0f : m[i];
#pragma unroll
        for (int r = 0; r < 4; ++r) ls[r] = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(fmaf(s[i][0][r], f[r >> 3], -mi2));
          s[i][0][r] = p;
          ls[r & 3] += p;
        }
      }
      l[i] += (ls[0] + ls[1]) + (ls[2] + ls[3]);
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
#pragma unroll
        for (int e = 0; e < 8; ++e) pf[i][k2][e] = (_Float16)s[i][0][8 * k2 + e];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      o[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[db].h, pf[0][0], o[0][db], 0, 0, 0);
      va[db].u = *reinterpret_cast<const uint4*>(vs + (32 * db + lrow) * kVStr + 16 + 8 * lh);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      o[0][db] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va[db].h, pf[0][1], o[0][db], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  if (first) store_tile(j & 1, vf0, vf1, nkf, nvf);
  __builtin_amdgcn_s_waitcnt(kWaitVm0);   // the direct K load
  __syncthreads();
  // Three loops (masked head, unmasked body, masked tail) rather than one
  // loop that picks the masked or unmasked tile per iteration: with both
  // variants in one loop body the compiler kept about 90 more registers
  // live.  Tiles past a row block's last row are fully masked for it and
  // skipped (only in the masked tail).
  // (A group's tiles alternate between its two buffers: KS is odd.)
  auto run_tiles = [&](int jb, auto mask_tag) __attribute__((always_inline)) {
    for (; j < jb; j += KS) {
      const bool more = j + KS < ntiles;
      u32x2 v0, v1;
      float nk, nv;
      if (more) {
        load_tile(j + KS, npage, kmem[(j + 1) & 1], v0, v1, nk, nv);
        npage = fetch_page(j + 2 * KS);
      }
      if (j < my_ntiles) tile(j, mask_tag);
      if (more) store_tile((j + 1) & 1, v0, v1, nk, nv);
      __builtin_amdgcn_s_waitcnt(kWaitVm0);
      __syncthreads();
    }
  };
  // the waves of the other row blocks stage nothing
  auto run_tiles_ns = [&](int jb, auto mask_tag) __attribute__((always_inline)) {
    for (; j < jb; ++j) {
      if (j < my_ntiles) tile(j, mask_tag);
      __syncthreads();
    }
  };
  if (stager) {
    run_tiles(min(ntiles, jlo), std::integral_constant<int, 2>{});
    run_tiles(nfull, std::integral_constant<int, 0>{});
    run_tiles(ntiles, std::integral_constant<int, 1>{});
  } else {
    run_tiles_ns(min(ntiles, jlo), std::integral_constant<int, 2>{});
    run_tiles_ns(nfull, std::integral_constant<int, 0>{});
    run_tiles_ns(ntiles, std::integral_constant<int, 1>{});
  }

  if constexpr (KS > 1) {
    // every group passes one barrier per tile of group 0
    if (j < j0 + kg + (ntiles - j0 + KS - 1) / KS * KS) __syncthreads();
    // weights 2^(m_g - M), M the row's maximum over the groups (0 for a group
    // that saw none of the row's keys); the outputs go through the V buffers,
    // 32 head dims at a time
    auto ml = reinterpret_cast<float (*)[4][32][2]>(&rl[0][0][0]);
    const float lw = l[0] + __shfl_xor(l[0], 32);
    if (lh == 0) {
      ml[kg][w][lrow][0] = m[0];
      ml[kg][w][lrow][1] = lw;
    }
    __syncthreads();
    float mx = -INFINITY, lt = 0.0f;
#pragma unroll
    for (int i = 0; i < KS; ++i) mx = fmaxf(mx, ml[i][w][lrow][0]);
#pragma unroll
    for (int i = 0; i < KS; ++i) {
      // a group that saw none of the row's keys adds nothing; one whose scores
      // are all NaN has no maximum either, but its sum is NaN
      const float mi = ml[i][w][lrow][0], li = ml[i][w][lrow][1];
      lt += mi == -INFINITY && li == 0.0f ? 0.0f : li * __builtin_amdgcn_exp2f(mi - mx);
    }
    const float f = m[0] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m[0] - mx);
    m[0] = mx;
    l[0] = lt;
    float4* xb = reinterpret_cast<float4*>(&vlds[0][0][0]);   // [group - 1][wave][4][64]
#pragma unroll
    for (int db = 0; db < 4; ++db) {
      if (db) __syncthreads();
      if (kg > 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          xb[(((kg - 1) * 4 + w) * 4 + i) * 64 + lane] =
              make_float4(o[0][db][4 * i] * f, o[0][db][4 * i + 1] * f,
                          o[0][db][4 * i + 2] * f, o[0][db][4 * i + 3] * f);
      }
      __syncthreads();
      if (kg == 0) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 a = xb[(w * 4 + i) * 64 + lane], b = xb[((4 + w) * 4 + i) * 64 + lane];
          o[0][db][4 * i] = fmaf(o[0][db][4 * i], f, a.x) + b.x;
          o[0][db][4 * i + 1] = fmaf(o[0][db][4 * i + 1], f, a.y) + b.y;
          o[0][db][4 * i + 2] = fmaf(o[0][db][4 * i + 2], f, a.z) + b.z;
          o[0][db][4 * i + 3] = fmaf(o[0][db][4 * i + 3], f, a.w) + b.w;
        }
      }
    }
    if (kg > 0) return;
  }

  // ---- epilogue
#pragma unroll
  for (int i = 0; i < HPW; ++i) {
    if (!wave_active[i]) continue;
    const float lt = KS > 1 ? l[i] : l[i] + __shfl_xor(l[i], 32);
    const int n_mine = min(32, it.n_rows - rbase);   // this row block's rows
    if (n_mine <= 0) continue;
    const int hq = g * G + (G >= 4 ? it.head0 : 0) + w + 4 * i;
    // lse (natural log) = (m + log2 l) * ln 2 with m in log2 units
    if (lse && lh == 0 && lrow < n_mine)
      lse[(int64_t)row * n_q_heads + hq] = (m[i] + log2f(lt)) * 0.69314718055994531f;
    // (the cos/sin rows' LDS is free: every wave is past a later barrier)
    static_assert(4 * R * kOutLds <= (int)sizeof(rl), "outputs go through it");
    store_out(o[i], 1.0f / lt, reinterpret_cast<uint8_t*>(&rl[0][0][0]) + (4 * rb + w) * kOutLds,
              lane, n_mine, out, [&](int r) -> int64_t {
                const int cr =
                    it.crow0 >= 0 ? it.crow0 + rbase + r : arows[it.row0 + rbase + r].row;
                return ((int64_t)cr * n_q_heads + hq) * kD;
              });
  }
}

int ilog2(int x) {
  int l = 0;
  while ((1 << l) < x) ++l;
  return l;
}

}  // namespace

hipError_t launch_attn_e4m3(const tsr_plan* p, const AttnItem* items, int32_t n_items,
                            const void* q, const void* req_k,
                            const void* req_v, const float* req_scale, void* out,
                            float* lse, hipStream_t s) {
  if (n_items == 0 || p->T == 0) return hipSuccess;
  const tsr_model& m = p->model;
  const int lp = ilog2(m.page_size);
  const int G = m.n_q_heads / m.n_kv_heads;
  const float sl2e = (float)((double)p->scale * 1.4426950408889634);
#define TSR_FP8(GG)                                                                   \
  if (p->row_blocks == kMaxRowBlocks)                                                 \
    TSR_FP8_R(GG, kMaxRowBlocks, 1);                                                  \
  else if (p->wave_groups == kWaveGroups)                                             \
    TSR_FP8_R(GG, 1, kWaveGroups);                                                    \
  else                                                                                \
    TSR_FP8_R(GG, 1, 1)
#define TSR_FP8_R(GG, RB, KS)                                                         \
  hipLaunchKernelGGL((attn_fp8_kernel<GG, RB, KS>), dim3(n_items), dim3(256 * (RB) * (KS)), \
                     0, s, static_cast<const uint16_t*>(q),                           \
                     static_cast<const uint8_t*>(req_k),                              \
                     static_cast<const uint8_t*>(req_v), req_scale, items,            \
                     p->dev.block_tables, p->dev.attn_rows, p->dev.rope_cos,          \
                     p->dev.rope_sin, static_cast<uint16_t*>(out), lse, m.n_q_heads,  \
                     m.n_kv_heads, lp, sl2e)
  switch (G) {
    case 1: TSR_FP8(1); break;
    case 2: TSR_FP8(2); break;
    case 4: TSR_FP8(4); break;
    case 8: TSR_FP8(8); break;
    default: return hipErrorInvalidValue;
  }
#undef TSR_FP8
#undef TSR_FP8_R
  return hipGetLastError();
}

}  // namespace tsr
