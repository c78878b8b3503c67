// Plans and workspace of the verify-token pass (gfx950), and the kernels that every pipeline
// shares: the reward head, the cache packing and the streaming read. The projections and the
// attention live in kvprm_mfma.hip and kvprm_attn.hip (bf16 weights) and kvprm_f32.hip (fp32).
#include <math.h>

#include <algorithm>

#include "kvprm_internal.h"
#include "kvprm_mx_common.h"

namespace kvprm {

// ------------------------------------------------------------------------------- plan

// Split-K plan of a matrix-core GEMV, in whole 32-wide input blocks: about 32 blocks per wave
// (long contiguous weight streams), but at least ~2048 waves in all and at least 4 blocks per
// slice. With one operand column tile the slice's operand is staged in LDS (1 KiB per block,
// <= 32 KiB); with more tiles the kernel reads it from memory.
static GemvPlan gemv_plan(int rows, int K, int B) {
  GemvPlan g;
  g.rows = rows;
  g.K = K;
  const int nt = gemv_nt(B);
  const int mt = gemv_mt(nt, rows);
  const int waves = (rows / 16 + mt - 1) / mt;
  const int nkb = K / 32;
  int want = (nkb + 31) / 32;
  const int want_par = (2048 + waves - 1) / waves;
  if (want < want_par) want = want_par;
  if (want > nkb / 4) want = nkb / 4;
  if (want < 1) want = 1;
  const int kb_per = (nkb + want - 1) / want;  // <= 32 unless the slice count is capped
  g.kslice = kb_per * 32;
  g.ksplit = (K + g.kslice - 1) / g.kslice;
  return g;
}

// Split-K plan of k_resid_split (wpb row tiles per block, batches of U input blocks): as many
// input slices as leave about one block per compute unit, each slice a whole number of batches.
static GemvPlan resid_split_plan(int rows, int K, int wpb, int U) {
  GemvPlan g;
  g.rows = rows;
  g.K = K;
  const int groups = (rows / 16 + wpb - 1) / wpb;
  const int nkb = K / 32;
  int want = 256 / groups;
  if (want < 1) want = 1;
  const int kb_per = ((nkb + want - 1) / want + U - 1) / U * U;
  g.kslice = kb_per * 32;
  g.ksplit = (nkb + kb_per - 1) / kb_per;
  return g;
}

static size_t partial_elems(const GemvPlan &g) {
  return (size_t)((g.ksplit + 3) & ~3) * g.rows;
}

// Bytes of keys and values of one page and head.
static int page_bytes(const Dims &dm) {
  return 2 * kPage * dm.d * (dm.kvdt == 0 ? 4 : dm.kvdt == 1 ? 2 : 1);
}

// Waves (kv-head x chunk) up to which shorter attention chunks pay: a wave takes about 4 us to
// start and end and 0.7 us per page pair however idle the chip is, so a small batch is fastest
// in many short chunks, until the waves' fixed cost and the merge's partials outweigh it; smaller tiles
// take more waves to load the memory system. 525 attention batches (six head layouts, bf16 and fp8, 1 to 64
// candidates of up to 32k tokens, equal, ragged and very ragged), distance from each one's fastest
// chunk length by this limit:
//   8 KiB of keys and values per page and head (bf16, d_h = 128)  500 1.8%, 600 1.0, 680 0.8, 800 1.7
//   4 KiB (bf16, 64; fp8, 128)                                     900 1.7%, 1000 1.2, 1100 1.4, 1280 2.3
//   2 KiB (fp8, 64)                                                2200 3.4%, 2560 1.5, 2850 0.9, 3600 2.4
// An fp32 page costs several times the products of a bf16 one (0.6 us at d_h = 64), so fp32
// chunks are shorter: up to two waves per SIMD unit.
static long long chunk_wave_limit(const Dims &dm) {
  if (dm.kvdt == 0) return 2048;
  const int bytes = page_bytes(dm);
  return bytes >= 8192 ? 680 : bytes >= 4096 ? 1080 : 2850;
}

int long_chunk_shift(long long pages) {
  int sh = 6;
  while (sh > 4 && pages < (160LL << sh)) --sh;
  return sh;
}

// The shortest chunk of 4, 8, .. 64 pages (fp32: 2 .. 32) whose waves stay within chunk_wave_limit and
// whose chunks fit the slots (kFineChunks below 16 pages); the longest otherwise. Without host
// lengths (known = false) the pages are those of a full table, more than the candidates hold, so that
// chunks are no longer than a full table's long ones. Chunk
// kernel alone: 1103 tokens x 8 heads 4.9 us (24.7 in 16-page chunks); 4096 tokens x 4
// heads 5.1 (16.2); four candidates of 4k-8k 11.8 (17.7).
// A wave is a block of its own, so that the work spreads over the compute units, except where 64-page
// chunks with all of 4 or more kv-heads in one block (whose tiles of a page are contiguous) fill most
// of one or two rounds of the chip, a block to each compute unit. The same 525 batches, all heads in a block
// against one: 13-18% slower at any chunk length, 1.4% faster on the 63 that this rule picks; eight of
// 200616 tokens in all, 4 heads 70.0 against 78.4 us a call (as waves of their own some units get four,
// others two or three), but 24 of 4096, 8 heads 96.5 against 65.1.
PrivateChunks private_chunk_rule(const Dims &dm, int n, const int *pages, const int *slots,
                                 bool known) {
  const bool f32 = dm.kvdt == 0;
  const int lo = f32 ? 1 : 2, hi = f32 ? 5 : 6;
  PrivateChunks r{hi, 1};
  long long total = 0, items = 0;
  for (int i = 0; i < n; ++i) total += pages[i];
  for (int sh = lo; sh <= hi; ++sh) {
    bool fits = true;
    items = 0;
    for (int i = 0; i < n; ++i) {
      const int ch = (pages[i] + (1 << sh) - 1) >> sh;
      items += ch;
      if (ch > slots[i] || (sh < 4 && ch > kFineChunks)) fits = false;
    }
    if (items * dm.nkv <= chunk_wave_limit(dm) && fits) {
      r.shift = sh;
      break;
    }
  }
  if (f32) return r;
  if (!known) {
    r.shift = std::min(r.shift, long_chunk_shift(total));
  } else if (r.shift == hi && dm.nkv >= 4) {
    const long long round = items <= 256 ? 256 : 512;
    if (items <= 512 && items * 10 >= round * 7) r.heads_per_block = dm.nkv;
  }
  return r;
}

// The backward attention runs eight waves (chunks) to a block and one block per compute unit
// (LDS), so that up to 2048 waves run at once; the chunk is the shortest of 2, 4, 8, 16 pages that
// keeps to that (a page takes a wave 4-5 us). Per layer, 7B shape: one candidate of 6000 tokens
// 74.9 us in 16-page chunks, 19.2 in 2; four of 4k-8k 82.3 -> 36.6 in 4; eight of 4k-8k
// 98.5 -> 65.2 in 8; eight of 16k-32k 275.6 in 16 (280.7 in 4).
constexpr long long kBackwardWaves = 2048;
int backward_chunk_pages(const Dims &dm, int n, const int *pages, int slots) {
  for (int CP = 2; CP < 16; CP *= 2) {
    long long items = 0;
    bool fits = true;
    for (int i = 0; i < n; ++i) {
      const int ch = (pages[i] + CP - 1) / CP;
      items += ch;
      if (ch > slots) fits = false;
    }
    if (fits && items * dm.nkv <= kBackwardWaves) return CP;
  }
  return 16;
}

Plan make_plan(const Dims &dm, int Breal, int max_pages, int lora_rank, int depth, bool lean) {
  Plan p{};
  const int B = Breal * depth;  // rows of the pass (verify tokens of all candidates)
  p.B = B;
  p.Breal = Breal;
  p.kq = depth;
  p.max_pages = max_pages;
  p.lora_rank = lora_rank;
  // chunk slots: chunks of max_pages at 16 pages (a long batch's chunks are no shorter) plus one
  // (a shared prefix that ends inside a chunk adds one), for whichever attention path runs; more
  // where the batch is small enough for shorter chunks (private_chunk_rule).
  // (fp32: 32-page chunks and shorter.) The room for all candidates' slots is a bound that never
  // falls with the batch or max_pages, so that a workspace serves every smaller batch too.
  const int longest = dm.kvdt == 0 ? kChunkPagesF32 : 16, shortest = dm.kvdt == 0 ? 2 : 4;
  p.nch = (max_pages + longest - 1) / longest + 1;
  p.slots = (size_t)Breal * p.nch;
  // the backward attention's: 16-page chunks, shorter for a small batch (backward_chunk_pages)
  p.nch_bwd = (max_pages + 15) / 16;
  p.slots_bwd = (size_t)Breal * p.nch_bwd;
  if (!lean) {
    auto fine = [&](long long waves, long long most, int *n, size_t *slots, int more) {
      const long long total = waves / dm.nkv, each = std::min(most, total / Breal) + more;
      if (*n < each) *n = (int)each;
      *slots = std::max(*slots, (size_t)(std::min(total, Breal * most) + (long long)Breal * more));
    };
    fine(chunk_wave_limit(dm), std::min(kFineChunks, (max_pages + shortest - 1) / shortest), &p.nch,
         &p.slots, 1);
    fine(kBackwardWaves, (max_pages + 1) / 2, &p.nch_bwd, &p.slots_bwd, 0);
  }
  size_t m = 0;
  if (dm.wdt == 1) {
    // split-K partials: the adapter's A-factor products and the split projections
    p.nt = gemv_nt(B);
    p.bp = gemv_bp(B);
    if (lora_rank > 0) {
      // A-factor products: rows = adapter rank per segment, input = the group's input width
      p.g_la[LORA_QKV] = gemv_plan(3 * lora_rank, dm.H, B);
      p.g_la[LORA_O] = gemv_plan(lora_rank, dm.nq * dm.d, B);
      p.g_la[LORA_GU] = gemv_plan(2 * lora_rank, dm.H, B);
      p.g_la[LORA_DOWN] = gemv_plan(lora_rank, dm.F, B);
      for (const GemvPlan &g : p.g_la) m = partial_elems(g) > m ? partial_elems(g) : m;
    }
    // the fused q/k/v kernel has one block per rotary tile pair; with more pairs than compute
    // units (320 at H = 8192, 64/8 heads) a second round leaves most of the chip idle, and the
    // split-K product with its finish kernel measured faster (28.3 vs 29.1 ms per call there)
    const int pairs = (dm.nq + 2 * dm.nkv) * (dm.d / 32);
    if (pairs > 256 && lora_rank == 0) {
      p.qkv_split = 1;
      p.g_qkv = gemv_plan((dm.nq + 2 * dm.nkv) * dm.d, dm.H, B);
      m = partial_elems(p.g_qkv) > m ? partial_elems(p.g_qkv) : m;
    }
    // Split-K projections (k_resid_split + a finish kernel): a fused kernel's block owns whole
    // rows over the whole input and reads the whole operand (NT KiB per input block) from L2,
    // for H / 16 row tiles (224 at the 7B shape, under one block per compute unit); the split
    // blocks share each operand batch over 8 row tiles and cover all compute units, at the cost
    // of one more launch. Measured per call: the down projection (ragged
    // 32k 4.79-4.82 -> 4.73-4.76 ms, 7B batch of 16 3.86 -> 3.59); output and q/k/v too for 9-16 rows
    // with at least 512 row tiles (large fp8 24.6 -> 23.7) and for more than 16 rows (beam
    // 7.92 -> 6.74 with output and down, 6.8 -> 6.75 with q/k/v). Short products lose more to the
    // second launch (3 to 4 us) than they gain. By how much the fused kernel is faster (-: slower),
    // us a layer, mean of eager and replayed calls of 2 to 28 layers, spread up to 1:
    //   down, inputs F      1024        2048        4096        8192        16384
    //   1-8 rows, H = 256   2.2..2.8    0.5..1.0    -1.1..-1.8  -4.1..-5.0  -10.5..-11.7
    //             H = 512   3.3..3.8    2.5..3.1    -0.2..0.4   -2.9..-3.9  -9.3..-10.0
    //             H = 1024  3.3..4.0    2.6..3.2    0.3..1.0    -1.8..-3.0  -6.9..-8.2
    //             H = 2048  2.9..4.0    2.1..3.5    0.1..1.9    0.5..1.7    -1.8..0.8
    //             H = 3072  2.9..3.9    2.2..3.3    0.3..1.1    0.1..1.3    -3.8..0.3
    //             H = 4096  3.5..3.8    2.0..2.7    1.7..3.0    2.8..3.7    2.5..3.4
    //   16 rows, any H      0.9..2.7    0.1..2.4    -2.1..2.7   -6.5..2.2   -16.0..-0.7
    //   48 rows, any H      0.7..4.1    -2.0..3.7   -8.2..0.7   -18..-4     -41..-18
    //   (H = 3584, 5120, 8192 with 18944, 17408, 28672 inputs, 1-8 rows: -1.9..-3.0, -11, -5..-7)
    //   q/k/v, up to 256 rotary tile pairs, 30 shapes of 24 to 48 heads:
    //   inputs H            2048        2560        3072        3584        4096        5120
    //   1-8 rows            0.9..2.8    0.5..2.1    1.8..2.9    0.9..2.8    0.7..2.8    2.5..3.8
    //   9-16 rows           -0.6..4.2   -1.3..0.8   0.4..4.2    -1.2..2.9   -1.9..2.5   -0.7..3.2
    //   17-64 rows          -0.3..5.1   -1.3..3.2   -2.4..1.2   -3.2..1.5   -4.4..0.9   -7.1..-1.3
    //   (smaller H: faster at all rows, 1.4..6.7.) More pairs than compute units take a second round of
    //   blocks: H = 8192, 320 pairs -7 at 9 rows, -35 at 64.
    // The output projection has fewer than 1024 inputs (H = 256: 33.9 / 40.2 at 32 rows fused / split).
    {
      // input blocks per batch of k_resid_split; with one column tile 16 where the input widths
      // divide (ragged 32k 4.75 -> 4.69 ms per call against 8), else 8
      int U = 4;
      if (p.nt == 1) U = (dm.nq * dm.d / 32) % 16 == 0 && (dm.F / 32) % 16 == 0 ? 16 : 8;
      const int down_fused = p.nt >= 4 ? 1024 : p.nt == 2 ? 2048  // inputs up to which it pays
                             : dm.H >= 2048 ? 8192 : dm.H >= 512 ? 4096 : 2048;
      const bool down = dm.F > down_fused;
      const bool out = p.nt >= 4 ? dm.nq * dm.d >= 1024 : p.nt == 2 && dm.H / 16 >= 512;
      const bool qkv = pairs > 256 ? p.nt >= 2 : p.nt >= 4 && dm.H >= 3072;
      if ((dm.nq * dm.d / 32) % U == 0 && (dm.F / 32) % U == 0) {
        // (8 row tiles per block measured faster than 16: 6.74 against 6.79 ms per call of the
        // 64-candidate beam)
        p.rs_wpb = 8;
        p.rs_u = U;
        p.rs_d = down;
        p.rs_o = out;
        p.g_rs_o = resid_split_plan(dm.H, dm.nq * dm.d, p.rs_wpb, U);
        p.g_rs_d = resid_split_plan(dm.H, dm.F, p.rs_wpb, U);
        if (qkv && (dm.H / 32) % U == 0 && (dm.nq + 2 * dm.nkv) * (dm.d / 2) >= 64) {
          p.rs_qkv = 1;
          p.g_rs_qkv = resid_split_plan((dm.nq + 2 * dm.nkv) * dm.d, dm.H, p.rs_wpb, U);
        }
        for (const GemvPlan *g : {&p.g_rs_o, &p.g_rs_d, &p.g_rs_qkv}) {
          // (with an adapter, one more slice: its B-factor tail)
          const size_t e = (size_t)(g->ksplit + (lora_rank > 0 ? 1 : 0)) * g->rows;
          m = e > m ? e : m;
        }
      }
    }
  }
  p.nss = dm.H / 16;  // (H is a multiple of 64)
  p.part_elems = m * (size_t)B;
  return p;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

Workspace carve(const Dims &dm, const Plan &p, void *base) {
  Workspace w{};
  char *c = (char *)base;
  size_t off = 0;
  auto take = [&](size_t elems) {
    float *r = base ? (float *)(c + off) : nullptr;
    off += align256(elems * sizeof(float));
    return r;
  };
  const size_t B = (size_t)p.B;
  w.x = take(B * dm.H);
  w.ss = take((size_t)p.nss * B);
  w.part = take(p.part_elems);
  w.q = take(B * dm.nq * dm.d);
  w.kself = take(B * dm.nkv * dm.d);
  w.vself = take(B * dm.nkv * dm.d);
  w.apart = take(p.slots * p.kq * dm.nq * (dm.d + 2));
  w.o = take(B * dm.nq * dm.d);
  w.hffn = take(B * dm.F);
  if (dm.wdt == 1) {
    const size_t per_k = (size_t)p.nt * 64 * 8 / 32;  // bf16 elements per input of an operand
    w.rope = take(B * dm.d);
    w.opA = (uint16_t *)take((per_k * dm.H + 1) / 2);
    w.opO = (uint16_t *)take((per_k * dm.nq * dm.d + 1) / 2);
    w.opD = (uint16_t *)take((per_k * dm.F + 1) / 2);
    if (p.lora_rank > 0) w.topd = (uint16_t *)take((per_k * 3 * p.lora_rank + 1) / 2);
  }
  if (dm.wdt == 0) {
    w.u = take(B * dm.H);
    w.rope64 = (double *)take(2 * B * dm.d);
  }
  w.bytes = off;
  return w;
}

// Workspace of the backward pass, after the forward's (see GradSave).
GradSave carve_grad(const Dims &dm, const Plan &p, void *base) {
  GradSave g{};
  char *c = (char *)base;
  size_t off = 0;
  auto take = [&](size_t elems) {
    float *r = base ? (float *)(c + off) : nullptr;
    off += align256(elems * sizeof(float));
    return r;
  };
  const size_t B = (size_t)p.B, NL = (size_t)dm.layers, H = dm.H, F = dm.F, d = dm.d;
  const size_t nq = dm.nq, nkv = dm.nkv;
  g.x_in = take(NL * B * H);
  g.x_mid = take(NL * B * H);
  g.q = take(NL * B * nq * d);
  g.ks = take(NL * B * nkv * d);
  g.vs = take(NL * B * nkv * d);
  g.o = take(NL * B * nq * d);
  g.lse = take(NL * B * nq);
  g.gu = take(NL * B * 2 * F);
  g.dx = take(B * H);
  g.dxT = take(kDPad * H);
  g.dxm = take(B * H);
  g.dxmT = take(kDPad * H);
  g.du = take(B * H);
  g.dgu = take(2 * F * kDPad);
  g.dout = take(B * nq * d);
  g.scores = take(B);
  g.dqkv = take((nq + 2 * nkv) * d * kDPad);
  g.dq_part = take(p.slots_bwd * nq * d);
  // split partials of the four transposed products
  size_t part = 0;
  const size_t cand[4][2] = {{F, H / 16}, {H, 2 * F / 16}, {nq * d, H / 16},
                             {H, (nq + 2 * nkv) * d / 16}};
  for (const auto &kt : cand) {
    const size_t n = (size_t)grad_tgemv_splits((int)kt[0], (int)kt[1]) * B * kt[0];
    part = n > part ? n : part;
  }
  g.part = take(part);
  g.bytes = off;
  return g;
}

// ------------------------------------------------------------------------------- attention

hipError_t launch_attention(const Dims &dm, const Plan &p, const Workspace &w, int layer,
                            const void *kpool, const void *vpool, const float *kscale,
                            const float *vscale, int num_pages, const int32_t *page_table,
                            const int32_t *lengths, const GroupTable &gt, const float *q,
                            const float *kself, const float *vself, float *o, uint16_t *op,
                            hipStream_t s, float *lse, bool partials_only) {
  const int EB = dm.kvdt == 0 ? 4 : (dm.kvdt == 1 ? 2 : 1);
  const size_t layer_elems = (size_t)num_pages * dm.nkv * kPage * dm.d;
  const char *kp = (const char *)kpool + layer_elems * EB * layer;
  const char *vp = (const char *)vpool + layer_elems * EB * layer;
  const float *ksc = kscale ? kscale + (size_t)layer * num_pages * dm.nkv : nullptr;
  const float *vsc = vscale ? vscale + (size_t)layer * num_pages * dm.nkv : nullptr;
  if (gt.one_launch && !partials_only)
    return launch_attn_short(dm, p, w, kp, vp, ksc, vsc, page_table, lengths, gt, q, kself, vself,
                             o, op, lse, s);
  hipError_t e =
      dm.kvdt == 0
          ? launch_attn_f32(dm, p, w, (const float *)kp, (const float *)vp, page_table, lengths, gt, q, s)
          : launch_attn_mx(dm, p, w, kp, vp, ksc, vsc, page_table, lengths, gt, q, s);
  if (e != hipSuccess || partials_only) return e;
  return launch_merge_mx(dm, p, w, lengths, gt, q, kself, vself, o, op, s, lse);
}

// ------------------------------------------------------------------------------- reward head

// z_b = w_r . (x_b / sqrt(mean(x_b^2) + eps) * gamma_f) + b_r; P(+) = sigmoid(z_b). One pass
// over x_b: sum(x^2) and sum(x gamma_f w_r) together (the RMS scale is a common factor of the
// dot product). One block per candidate, so the kernel is one memory round trip and a reduction:
// 1024 threads with eight elements each in flight (256 threads walking the row took 9.4 us at
// H = 3584 and 18.8 at 8192; now 4.5 and 7.0).
constexpr int kHeadThreads = 1024;
__global__ __launch_bounds__(kHeadThreads) void k_head(const float *x, int H, float eps,
                                                       const void *gam, const void *wr, int wdt,
                                                       float rb, float *scores, float *logits,
                                                       int kq) {
  constexpr int U = 8, NW = kHeadThreads / 64;
  __shared__ float red[2][NW];
  const int b = blockIdx.x;
  const float *xb = x + ((size_t)b * kq + kq - 1) * H;  // the candidate's last verify token
  float sq = 0.f, dot = 0.f;
  for (int r0 = threadIdx.x; r0 < H; r0 += U * kHeadThreads) {
    float v[U], gv[U], wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r0 + u * kHeadThreads < H) {
        v[u] = xb[r0 + u * kHeadThreads];
        gv[u] = ld_w(gam, r0 + u * kHeadThreads, wdt);
        wv[u] = ld_w(wr, r0 + u * kHeadThreads, wdt);
      } else {
        v[u] = gv[u] = wv[u] = 0.f;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      sq += v[u] * v[u];
      dot += v[u] * (gv[u] * wv[u]);
    }
  }
  sq = wsum(sq);
  dot = wsum(dot);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = sq;
    red[1][threadIdx.x >> 6] = dot;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    sq = dot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      sq += red[0][w];
      dot += red[1][w];
    }
    const float inv = 1.0f / sqrtf(sq / (float)H + eps);
    const float z = dot * inv + rb;
    float pz;
    if (z >= 0.f) {
      pz = 1.0f / (1.0f + expf(-z));
    } else {
      const float ez = expf(z);
      pz = ez / (1.0f + ez);
    }
    scores[b] = pz;
    if (logits) logits[b] = z;
  }
}

hipError_t launch_head(const Dims &dm, const Plan &p, const Workspace &w, const void *final_norm,
                       const void *reward_w, float reward_b, float *scores, float *logits,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_head, dim3(p.Breal), dim3(kHeadThreads), 0, s, w.x, dm.H, dm.eps, final_norm,
                     reward_w, dm.wdt, reward_b, scores, logits, p.kq);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------- cache packing

// 16 bytes that a call writes once: non-temporal, as ld_stream
__device__ __forceinline__ void st_once(uint4 *p, const uint4 &v) {
  __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), (u32x4 *)p);
}

// Token-major cache tiles ([page_size][d] values, slot-major) -> the stored K or V tile layout.
// One block per 4 KiB of tiles, or per tile where that is larger (grid-stride): the tiles are read
// into LDS with 16-byte loads, then every thread assembles 16-byte output groups in output order
// and stores them, so both the reads and the writes are contiguous and a small tile (1 KiB: fp8,
// d_h = 64) leaves no thread of the block without work. EB = element bytes; x = 16 / EB values per group.
// The tile size is a template argument: computed from d at run time it cost 4 KiB tiles 3% (4 layers of
// 8000 tokens, 7B shape, 41 MB a part: 26.3 us for both parts, 25.3 so).
//   K group (m / x) * 16 + s holds dims m .. m + x - 1 of slot s (a contiguous source run);
//   V group ((m / (16 r)) * 4 + s / 4) * 16 + m % 16 holds slots 4 (s / 4) .. + 3 of the r dims
//   m % 16 + 16 i (i < r) of the 16 r-dim block, as [i][slot % 4] (r = x / 4).
template <int EB, int D, bool V, bool ONCE>
__global__ __launch_bounds__(256) void k_pack_kv(const uint4 *__restrict__ src, uint4 *__restrict__ dst,
                                                 int64_t ntiles) {
  constexpr int X = 16 / EB, R = X / 4;
  constexpr int groups = D * EB;  // 16-byte groups per tile (64 to 512, a power of two)
  constexpr int per = groups < 256 ? 256 / groups : 1;  // tiles at a time
  __shared__ uint4 tile_s[per * groups];
  for (int64_t t0 = (int64_t)blockIdx.x * per; t0 < ntiles; t0 += (int64_t)gridDim.x * per) {
    const int n = (int)(ntiles - t0 < per ? ntiles - t0 : per) * groups;
    const uint4 *sp = src + t0 * groups;
    for (int i = threadIdx.x; i < n; i += 256) tile_s[i] = ONCE ? ld_stream(sp + i) : sp[i];
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 256) {
      const int gi = i & (groups - 1);
      const uint4 *ts = tile_s + (i - gi);
      uint4 out;
      if (!V) {
        const int s = gi & 15, mb = gi >> 4;  // slot, x-dim block
        out = ts[s * (D / X) + mb];
      } else {
        const unsigned char *tb = (const unsigned char *)ts;
        const int mm = gi & 15, sq = (gi >> 4) & 3, blk = gi >> 6;
        unsigned char *ob = (unsigned char *)&out;
#pragma unroll
        for (int q = 0; q < R; ++q)
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const int m = blk * 16 * R + q * 16 + mm, sl = 4 * sq + k;
#pragma unroll
            for (int e = 0; e < EB; ++e) ob[(q * 4 + k) * EB + e] = tb[(sl * D + m) * EB + e];
          }
      }
      if (ONCE)
        st_once(dst + t0 * groups + i, out);
      else
        dst[t0 * groups + i] = out;
    }
    __syncthreads();
  }
}

hipError_t launch_pack_kv(const void *src, void *dst, int64_t ntiles, int d, int eb, bool v,
                          hipStream_t s) {
  const int groups = d * eb, per = groups < 256 ? 256 / groups : 1;
  int64_t blocks = (ntiles + per - 1) / per;
  blocks = blocks < 65536 ? blocks : 65536;
  const dim3 grid((unsigned)blocks), block(256);
  const uint4 *a = (const uint4 *)src;
  uint4 *b = (uint4 *)dst;
  // Non-temporal from 128 MiB read and written: keys and values together then exceed the 256 MiB
  // memory-side cache, and leaving it alone is faster (28 layers of 8192 tokens at the 7B shape:
  // 194 -> 185 us for both parts, 180 with the tile size fixed at compile time); below, the packed tiles stay there for their first reader (4 layers
  // of 4000 fp32 tokens, 164 MB in all: 26.1 us plain, 29.6 non-temporal).
  const bool once = ntiles * (int64_t)groups * 32 >= (int64_t)128 << 20;
#define KVPRM_PK(E_, D_, V_)                                                                          \
  if (once) hipLaunchKernelGGL((k_pack_kv<E_, D_, V_, true>), grid, block, 0, s, a, b, ntiles);       \
  else hipLaunchKernelGGL((k_pack_kv<E_, D_, V_, false>), grid, block, 0, s, a, b, ntiles)
#define KVPRM_PKD(E_)                          \
  if (d == 64) {                               \
    if (v) { KVPRM_PK(E_, 64, true); }         \
    else { KVPRM_PK(E_, 64, false); }          \
  } else {                                     \
    if (v) { KVPRM_PK(E_, 128, true); }        \
    else { KVPRM_PK(E_, 128, false); }         \
  }
  if (d != 64 && d != 128) return hipErrorInvalidValue;
  switch (eb) {
    case 4: KVPRM_PKD(4); break;
    case 2: KVPRM_PKD(2); break;
    case 1: KVPRM_PKD(1); break;
    default: return hipErrorInvalidValue;
  }
#undef KVPRM_PKD
#undef KVPRM_PK
  return hipGetLastError();
}

// ------------------------------------------------------------------------------- diagnostics

// Streaming read of n16 16-byte words: grid-stride, four non-temporal loads in flight per
// thread, the words folded into an XOR that each wave adds to *sink with one atomic, so that the
// loads cannot be removed (and a test can check that every word was read once). The reference
// ceiling for the kernels' HBM fractions.
__global__ __launch_bounds__(256) void k_stream_read(const uint4 *buf, size_t n16, uint32_t *sink) {
  const size_t stride = (size_t)gridDim.x * 256;
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  uint32_t acc = 0;
  for (; i + 3 * stride < n16; i += 4 * stride) {
    u32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load((const u32x4 *)(buf + i + u * stride));
#pragma unroll
    for (int u = 0; u < 4; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; i < n16; i += stride) {
    const u32x4 v = __builtin_nontemporal_load((const u32x4 *)(buf + i));
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc ^= (uint32_t)__shfl_xor((int)acc, off, 64);
  if ((threadIdx.x & 63) == 0) atomicXor(sink, acc);
}

hipError_t launch_stream_read(const void *buf, size_t bytes, uint32_t *sink, hipStream_t s) {
  // 512 blocks of 4 waves: the fastest shape of a plain streaming read on this chip (256 blocks
  // leave the memory system short of requests, 1024 and more add contention)
  hipLaunchKernelGGL(k_stream_read, dim3(512), dim3(256), 0, s, (const uint4 *)buf, bytes / 16,
                     sink);
  return hipGetLastError();
}

}  // namespace kvprm
