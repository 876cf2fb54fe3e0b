// fp32 sparse branch with the linear branch and the gated fusion in the
// epilogue: the same path as the bf16 walks (Sec. 3.3 "Sparse branch", App.
// A.1 eq. attention) with fp32 operands, products and sums throughout.
//
// Both products run on the fp32 matrix instruction (16x16x4: a full fp32
// multiply and add per term, twice the work per cycle of VALU FMAs, and one LDS
// read per operand and tile where an FMA needs one per term). The scores are
// computed transposed, S^T = K Q^T, so that lane l holds four scores of query
// l % 16 per 16 keys, and the same registers are the B operand of O^T += V^T
// P^T: probabilities never leave their lane. The contraction order over d and
// over keys is free as long as both operands agree, so a lane's operands are
// four consecutive floats (16 bytes) of a key row or of a d-major value row.
//
// A work item is 64 queries of one (b, h): eight waves, 16 queries by one of
// two key streams each. The streams take alternate 32-key tiles and are merged
// through LDS at the end. The items' steps (64 keys) are laid end to end and
// cut into equal ranges, one per workgroup; an item that a range boundary cuts
// is merged by the last of its pieces to arrive, in piece order.
//
// Bound: the matrix pipes (4 n_q d per key and head; a large fp32 product
// reaches 154 TFLOP/s). A step of eight MFMAs reads 2 KB per wave, a quarter of
// the LDS bandwidth, and the tiles come from L2, so the tile loads go through
// registers, which takes pointers of any 4-byte alignment. Measured (8 heads x
// d128, 1170 queries, lists of 5 and 7 pages of 392 keys): 147 us, 77 TFLOP/s of
// the work, the matrix pipes busy 0.61 of the cycles at a 2.13 GHz clock; the
// VALU kernel before it took 3400 us. 2 heads x d64, 256 queries, 3 pages of
// 256: 17 us against 283.
#include <float.h>

#include <algorithm>
#include <cmath>

#include "hsa_device.h"
#include "hsa_kernels.h"

namespace hsa {
namespace {

constexpr int kQB = 64;    // queries per workgroup
constexpr int kTK = 32;    // keys per tile of one stream
constexpr int kWaves = 8;  // 4 query groups x 2 key streams

__device__ __forceinline__ f32x4 ld4s(const float* p) { return *reinterpret_cast<const f32x4*>(p); }

// D[16x16] += A[16x4] B[4x16]: lane l supplies A row l % 16 and B column
// l % 16 at k = l / 16; register r of lane l is row 4 (l / 16) + r, column l % 16.
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// LDS tiles in 16-byte chunks, XOR-swizzled so that 16 consecutive rows read
// at one logical chunk fall on all 64 banks: key rows of 4 D bytes, value rows
// (one d each) of 128 bytes. Indices in floats.
template <int D>
__device__ __forceinline__ int k_at(int row, int ch) { return row * D + ((ch ^ (row & 15)) << 2); }
__device__ __forceinline__ int v_at(int row, int ch) { return row * kTK + ((ch ^ ((row >> 1) & 7)) << 2); }

// Schedule of N steps of eight MFMAs, each on two 16-byte LDS reads: the
// reads of a step are issued in the middle of the step A before it.
template <int N, int A>
__device__ __forceinline__ void pipeline_steps() {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);                // MFMA
    if (i + A < N) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0); // LDS read
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
  }
}
template <int N, int A>
__device__ __forceinline__ void pipeline_reads() {
  __builtin_amdgcn_sched_group_barrier(0x100, 2 * A, 0);
  pipeline_steps<N, A>();
}

// Floats of one stream's tile (keys, then values); two buffers per stream.
template <int D>
constexpr int kTileF = 2 * kTK * D;

template <int D, bool kList>
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 4 : 2) void attn_f32_kernel(AttnParams p_arg) {
  constexpr int NM = D / 16, NH = NM / 2;     // 16-wide d blocks, of which a wave finishes half
  constexpr int NC = D / 16;                  // 16-wide slices of d in the score product
  constexpr int NLD = kTK * D / 4 / 256;      // 16-byte loads per thread, tile and tensor
  __shared__ __attribute__((aligned(16))) float smem[4 * kTileF<D>];
  // Workgroup ids go round-robin to the 8 XCDs; each XCD takes consecutive
  // ranges, so that neighbouring query blocks share their keys in its L2.
  // Ranges [0, sk_rm) hold sk_q + 1 steps, the others sk_q.
  auto range_id = [](const AttnSchedule& sc) {
    const int G = sc.sk_g, x = (int)(blockIdx.x & 7);
    return x * (G >> 3) + min(x, G & 7) + (int)(blockIdx.x >> 3);
  };
  auto range_start = [](const AttnSchedule& sc, int i) { return i * sc.sk_q + min(i, sc.sk_rm); };
  auto range_of = [](const AttnSchedule& sc, int t) {
    const int big = sc.sk_rm * (sc.sk_q + 1);
    return t < big ? t / (sc.sk_q + 1) : sc.sk_rm + (t - big) / sc.sk_q;
  };
  int t_seg = range_start(p_arg.sc, range_id(p_arg.sc));
  const int t_end = range_start(p_arg.sc, range_id(p_arg.sc) + 1);
  while (t_seg < t_end) {
  __syncthreads();  // the previous segment is done with the LDS
  // The segment reads the parameters (through the kernel-argument segment) and
  // the lane's index through values the compiler cannot see through: it would
  // otherwise hoist what only the epilogue needs out of the loop and keep it
  // live across the walk.
  using ArgParams = const __attribute__((address_space(4))) AttnParams;
  ArgParams* pa = (ArgParams*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(pa));
  const AttnParams& p = *(const AttnParams*)pa;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int s = wave >> 2, qg = wave & 3;     // key stream, query group
  const int l16 = lane & 15, g = lane >> 4;
  const int H = p.H, P = p.P, nqb = (p.n_q + kQB - 1) / kQB;
  const int per_b = p.sc.sk_head_off[H];
  const int b = t_seg / per_b, tb = t_seg - b * per_b;
  int h = 0;
  while (h + 1 < H && p.sc.sk_head_off[h + 1] <= tb) ++h;
  const int n_steps = (p.sc.sk_head_off[h + 1] - p.sc.sk_head_off[h]) / nqb;
  const int ih = tb - p.sc.sk_head_off[h];
  const int qb = ih / n_steps, seg_a = ih - qb * n_steps;  // this segment: steps [seg_a, seg_e) of the item
  const int item0 = t_seg - seg_a, seg_e = min(n_steps, t_end - item0);
  t_seg = item0 + seg_e;

  // ---- the item's tiles: 32-key tiles of the page list, or the entries
  // (64-key tiles) of the tile list; the segment takes its share of them (the
  // steps are planned from a bound on the list, which may be shorter)
  const int32_t* selrow = p.sel + ((size_t)b * H + h) * p.k_max;
  const int32_t* ptrow = p.page_table + (size_t)b * p.max_pages;
  const int tpp = (P + kTK - 1) / kTK;
  int n_sel = 0, total;
  const int2* lst = nullptr;
  const int bit = qb & 1;
  if constexpr (kList) {
    const size_t cell = ((size_t)b * H + h) * p.sc.nqt + qb / 2;
    total = ld_const(p.blist_len + cell);
    lst = p.blist + cell * p.blist_cap;
  } else {
    n_sel = count_selected(selrow, p.k_max, p.max_pages, lane);
    total = (n_sel + p.n_cur) * tpp;
  }
  int u = (int)((long)total * seg_a / n_steps);
  const int u_end = (int)((long)total * seg_e / n_steps);

  // The next tile of this stream at or after u: its (slot, head) row, first
  // key and the end of its keys in the page (k0 >= k1: none for this stream).
  // Both streams advance u alike, so the workgroup's trip counts agree.
  size_t ph = 0;
  int k0 = 0, k1 = 0, li_ph = -1;
  auto next_tile = [&]() -> bool {
    if constexpr (kList) {
      int2 e = make_int2(0, 0);
      while (u < u_end) {
        e = ld_const(lst + u);
        if ((e.y >> bit) & 1) break;
        ++u;
      }
      if (u >= u_end) return false;
      ++u;
      ph = (size_t)e.x;
      k0 = (e.y >> 2) * 64 + kTK * s;
      k1 = min(P, k0 + kTK);
    } else {
      if (u >= u_end) return false;
      const int t = u + s;
      u += 2;
      k0 = k1 = 0;
      if (t < u_end) {
        const int li = t / tpp;
        if (li != li_ph) {
          const int lp = li < n_sel ? ld_const(selrow + li) : p.cur_first + (li - n_sel);
          ph = (size_t)clampi(ld_const(ptrow + lp), 0, p.num_slots - 1) * H + h;
          li_ph = li;
        }
        k0 = (t - li * tpp) * kTK;
        k1 = min(P, k0 + kTK);
      }
    }
    return true;
  };

  // ---- tile loads: the 32-key window that ends at the page end when fewer
  // keys remain (rows before k0 are masked); pages shorter than a tile clamp
  const float* kg = static_cast<const float*>(p.k);
  const float* vg = static_cast<const float*>(p.v);
  const int ts = tid & 255;
  f32x4 kr[NLD], vr[NLD];
  auto load = [&]() {
    const int ws = max(0, min(k0, P - kTK));
    const float* kp = kg + ph * P * D;
    const float* vp = vg + ph * D * P;
#pragma unroll
    for (int n = 0; n < NLD; ++n) {
      const int x = ts + 256 * n, row = x / (D / 4), ch = x % (D / 4);
      kr[n] = ld4u(kp + (size_t)min(ws + row, P - 1) * D + 4 * ch);
    }
#pragma unroll
    for (int n = 0; n < NLD; ++n) {
      const int x = ts + 256 * n, row = x >> 3, ch = x & 7;
      vr[n] = ld4u(vp + (size_t)row * P + min(ws + 4 * ch, P - 4));
    }
  };
  // (value columns outside [k0, k1) are stored as zeros: their probabilities
  // are zero, and a zero times an infinite value would be NaN)
  auto store = [&](int buf) {
    const int ws = max(0, min(k0, P - kTK)), lo = k0 - ws, hi = k1 - ws;
    float* kt = smem + (2 * s + buf) * kTileF<D>;
    float* vt = kt + kTK * D;
#pragma unroll
    for (int n = 0; n < NLD; ++n) {
      const int x = ts + 256 * n;
      *reinterpret_cast<f32x4*>(kt + k_at<D>(x / (D / 4), x % (D / 4))) = kr[n];
    }
#pragma unroll
    for (int n = 0; n < NLD; ++n) {
      const int x = ts + 256 * n;
      const int key = 4 * (x & 7);  // lo and hi are multiples of 8
      *reinterpret_cast<f32x4*>(vt + v_at(x >> 3, x & 7)) = key >= lo && key < hi ? vr[n] : f32x4{0};
    }
  };

  bool have = next_tile();
  if (have && k0 < k1) load();

  // ---- query fragment: query l16 of the group, d = 16 c + 4 g + 0..3
  const int q_idx = qb * kQB + 16 * qg + l16;
  const bool q_ok = q_idx < p.n_q;
  f32x4 qf[NC];
  {
    const float* qrow = static_cast<const float*>(p.q) +
                        (((size_t)b * p.n_q + min(q_idx, p.n_q - 1)) * H + h) * D + 4 * g;
#pragma unroll
    for (int c = 0; c < NC; ++c) qf[c] = ld4u(qrow + 16 * c);
    // pinned here, the fragments count as loaded for the compiler; it would
    // otherwise wait for the walk's tile loads inside every score product
#pragma unroll
    for (int c = 0; c < NC; ++c) asm volatile("" : "+v"(qf[c]));
  }
  f32x4 acc[NM];
#pragma unroll
  for (int m = 0; m < NM; ++m) acc[m] = f32x4{0};
  const float c2 = p.scale_log2;
  float m_run = softmax_floor(c2), l_run = 0.f;

  // keys lo..hi-1 of the window in LDS buffer buf
  auto compute = [&](int buf, int lo, int hi) {
    const float* kt = smem + (2 * s + buf) * kTileF<D>;
    const float* vt = kt + kTK * D;
    // operands are read two steps (of eight MFMAs) ahead of their use
    constexpr int kAhead = 2;
    f32x4 a[kAhead][2];
    auto kop = [&](int c, f32x4 (&f)[2]) {
      f[0] = ld4s(kt + k_at<D>(l16, 4 * c + g));
      f[1] = ld4s(kt + k_at<D>(16 + l16, 4 * c + g));
    };
    auto vop = [&](int i, f32x4 (&f)[2]) {  // step i: keys 16 (i / NH).., d blocks 2 (i % NH), + 1
      const int kb = i / NH, m = 2 * (i % NH);
      f[0] = ld4s(vt + v_at(16 * m + l16, 4 * kb + g));
      f[1] = ld4s(vt + v_at(16 * m + 16 + l16, 4 * kb + g));
    };
    // Two partial sums per score, each over half of d: the instruction rounds
    // after every term, and one chain over d = 128 leaves twice the error (8
    // heads x d128, 1170 queries, a whole step: 195 us, with one chain 192).
    f32x4 sc[2] = {f32x4{0}, f32x4{0}}, sd[2] = {f32x4{0}, f32x4{0}};
#pragma unroll
    for (int c = 0; c < kAhead; ++c) kop(c, a[c]);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      f32x4 f[2] = {a[c % kAhead][0], a[c % kAhead][1]};
      if (c + kAhead < NC) kop(c + kAhead, a[c % kAhead]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f32x4 (&t)[2] = c < NC / 2 ? sc : sd;
        t[0] = mfma16(f[0][e], qf[c][e], t[0]);
        t[1] = mfma16(f[1][e], qf[c][e], t[1]);
      }
    }
    pipeline_reads<NC, kAhead>();
    sc[0] += sd[0];
    sc[1] += sd[1];
    __builtin_amdgcn_sched_barrier(0);
    f32x4 w[kAhead][2];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) vop(i, w[i]);
    if (lo > 0 || hi < kTK) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = 16 * kb + 4 * g + r;
          if (key < lo || key >= hi) sc[kb][r] = -INFINITY;
        }
    }
    // online softmax against a reference maximum that moves only when a score
    // exceeds it by more than 8 in log2 units (exact for any reference). Scores
    // are compared and subtracted before they are scaled: the difference is
    // small and exact where it matters, while a scaled score of 2^31 or more is
    // rounded by more than the exponent of a float can hold.
    float mx = fmaxf(fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3])),
                     fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
    if (__any((mx - m_run) * c2 > 8.f)) {
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const bool grow = (mx - m_run) * c2 > 8.f;
      const float m_new = grow ? mx : m_run;
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * c2);
      l_run *= alpha;
#pragma unroll
      for (int m = 0; m < NM; ++m) acc[m] *= alpha;
      m_run = m_new;
    }
    float pv[2][4];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 4; ++r) pv[kb][r] = __builtin_amdgcn_exp2f((sc[kb][r] - m_run) * c2);
    l_run += ((pv[0][0] + pv[0][1]) + (pv[0][2] + pv[0][3])) + ((pv[1][0] + pv[1][1]) + (pv[1][2] + pv[1][3]));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 2 * NH; ++i) {
      const int kb = i / NH, m = 2 * (i % NH);
      f32x4 f[2] = {w[i % kAhead][0], w[i % kAhead][1]};
      if (i + kAhead < 2 * NH) vop(i + kAhead, w[i % kAhead]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[m] = mfma16(f[0][r], pv[kb][r], acc[m]);
        acc[m + 1] = mfma16(f[1][r], pv[kb][r], acc[m + 1]);
      }
    }
    pipeline_steps<2 * NH, kAhead>();
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- walk: tile t + 1 is in flight (registers) while tile t, in LDS, is
  // computed; one barrier per step
  if (have && k0 < k1) store(0);
  lds_barrier();
  for (int buf = 0; have; buf ^= 1) {
    const int ws = max(0, min(k0, P - kTK)), lo = k0 - ws, hi = k1 - ws;
    const bool mine = k0 < k1;
    have = next_tile();
    if (have && k0 < k1) load();
    if (mine) compute(buf, lo, hi);
    if (have && k0 < k1) store(buf ^ 1);
    lds_barrier();
  }

  // ---- the two streams of a query group: each wave hands over the half of
  // the d blocks that its partner finishes, and both weigh them alike
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  f32x4 oa[NH];
  float m_tot, l_tot;
  {
    constexpr int W = (4 * NH + 2) * 64;   // floats of one wave's message
    float* out = smem + wave * W + lane;
    const float* in = smem + (wave ^ 4) * W + lane;
    out[0] = m_run;
    out[64] = l_run;
#pragma unroll
    for (int i = 0; i < NH; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(2 + 4 * i + r) * 64] = s ? acc[i][r] : acc[NH + i][r];
    lds_barrier();
    const float m_o = in[0], l_o = in[64];
    m_tot = fmaxf(m_run, m_o);
    const float w = __builtin_amdgcn_exp2f((m_run - m_tot) * c2);
    const float w_o = __builtin_amdgcn_exp2f((m_o - m_tot) * c2);
    const float w0 = s ? w_o : w, w1 = s ? w : w_o;   // weights of streams 0 and 1
    l_tot = s ? fmaf(w0, l_o, w1 * l_run) : fmaf(w0, l_run, w1 * l_o);
#pragma unroll
    for (int i = 0; i < NH; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float a = s ? acc[NH + i][r] : acc[i][r], o = in[(2 + 4 * i + r) * 64];
        oa[i][r] = s ? fmaf(w0, o, w1 * a) : fmaf(w0, a, w1 * o);
      }
  }

  // ---- pieces: every one leaves its sums, reference maximum and row sum in
  // its slot (written through to the device's point of coherence: the pieces
  // may run on XCDs whose L2 caches are not coherent), then counts itself in;
  // the last to arrive merges them all in piece order, four pieces' loads in
  // flight at a time. Piece k is range r_first + k's first segment (slot 0),
  // except for k = 0 when the item starts inside that range (its last, slot 1).
  const int r_first = range_of(p.sc, item0);
  const int np = range_of(p.sc, item0 + n_steps - 1) - r_first + 1;
  if (np > 1) {
    constexpr int W = (4 * NH + 2) * 64;
    const int slot0 = item0 != range_start(p.sc, r_first) ? 1 : 0;
    auto slot = [&](int k) {
      return p.part_o + ((size_t)((r_first + k) * 2 + (k == 0 ? slot0 : 0)) * kWaves + wave) * W + lane;
    };
    auto put = [](float* q, float v) { __hip_atomic_store(q, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    auto get = [](const float* q) { return __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    float* out = slot(range_id(p.sc) - r_first);
    put(out, m_tot);
    put(out + 64, l_tot);
#pragma unroll
    for (int i = 0; i < NH; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) put(out + (2 + 4 * i + r) * 64, oa[i][r]);
    wait_vmcnt<0>();
    __syncthreads();  // every wave's sums are out, and the messages in LDS are read
    int* s_last = reinterpret_cast<int*>(smem);
    if (tid == 0)
      *s_last = __hip_atomic_fetch_add(p.attn_ctr + ((size_t)b * H + h) * nqb + qb, 1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT) == np - 1;
    __syncthreads();
    if (!*s_last) continue;
    constexpr int kB = 4;
    m_tot = -INFINITY;
    for (int k = 0; k < np; k += kB) {
      float m4[kB];
#pragma unroll
      for (int j = 0; j < kB; ++j) m4[j] = get(slot(min(k + j, np - 1)));
#pragma unroll
      for (int j = 0; j < kB; ++j) m_tot = fmaxf(m_tot, m4[j]);
    }
    l_tot = 0.f;
#pragma unroll
    for (int i = 0; i < NH; ++i) oa[i] = f32x4{0};
    for (int k = 0; k < np; k += kB) {
      float m4[kB], l4[kB], v[kB][4 * NH];
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        const float* in = slot(min(k + j, np - 1));
        m4[j] = get(in);
        l4[j] = get(in + 64);
#pragma unroll
        for (int i = 0; i < 4 * NH; ++i) v[j][i] = get(in + (2 + i) * 64);
      }
#pragma unroll
      for (int j = 0; j < kB; ++j) {
        if (k + j >= np) break;
        const float w = __builtin_amdgcn_exp2f((m4[j] - m_tot) * c2);
        l_tot = fmaf(w, l4[j], l_tot);
#pragma unroll
        for (int i = 0; i < 4 * NH; ++i) oa[i / 4][i % 4] = fmaf(w, v[j][i], oa[i / 4][i % 4]);
      }
    }
  }

  // ---- epilogue: this wave's half of the rows of its 16 queries; lane holds
  // query l16, dims 16 m + 4 g + 0..3 of block m = s NH + i
  const float inv_l = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const size_t gi = ((size_t)b * p.n_q + q_idx) * H + h;
  if (p.mode == ATTN_SPARSE) {
    if (!q_ok) continue;
#pragma unroll
    for (int i = 0; i < NH; ++i) st4u(p.o_sp + gi * D + 16 * (s * NH + i) + 4 * g, oa[i] * inv_l);
    if (p.lse && s == 0 && g == 0)
      p.lse[((size_t)b * H + h) * p.n_q + q_idx] = l_tot > 0.f ? m_tot * p.sm_scale + logf(l_tot) : -INFINITY;
    continue;
  }
  // gate weights: one per (query, head), or per element with gate_elem
  auto sigm = [](float x) { return 1.f / (1.f + expf(-x)); };
  auto sig = [&](const float* gt, size_t i) { return gt ? sigm(gt[i]) : 0.5f; };
  float wl = 0.5f, wsp = 0.5f;
  if (q_ok && !p.gate_elem) {
    wl = sig(p.g_lin, gi);
    wsp = sig(p.g_sp, gi);
  }
  auto write = [&](int i, f32x4 lin) {  // lin: the linear branch's four values
    if (!q_ok) return;
    const size_t e0 = gi * D + 16 * (s * NH + i) + 4 * g;
    f32x4 gl = f32x4{0}, gs = f32x4{0}, o;
    if (p.gate_elem && p.g_lin) gl = ld4u(p.g_lin + e0);
    if (p.gate_elem && p.g_sp) gs = ld4u(p.g_sp + e0);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float a = p.gate_elem ? sigm(gl[r]) : wl, c = p.gate_elem ? sigm(gs[r]) : wsp;
      o[r] = a * lin[r] + c * oa[i][r] * inv_l;
    }
    st4u(static_cast<float*>(p.o) + e0, o);
  };
  if (p.o_lin) {  // linear branch from another launch (Linformer)
#pragma unroll
    for (int i = 0; i < NH; ++i)
      write(i, q_ok ? ld4u(p.o_lin + gi * D + 16 * (s * NH + i) + 4 * g) : f32x4{0});
    continue;
  }
  // O_lin^T = S phi(Q)^T / (phi(Q) . z)
  const float* st = p.kv_state + ((size_t)b * H + h) * D * D;
  const float* zz = p.k_state + ((size_t)b * H + h) * D;
  float den = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const f32x4 z = ld4u(zz + 16 * c + 4 * g);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      qf[c][e] = phi(qf[c][e]);
      den = fmaf(qf[c][e], z[e], den);
    }
  }
  den += __shfl_xor(den, 16);
  den += __shfl_xor(den, 32);
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    const float* row = st + (size_t)(16 * (s * NH + i) + l16) * D + 4 * g;
    f32x4 num = f32x4{0};
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const f32x4 a = ld4u(row + 16 * c);
#pragma unroll
      for (int e = 0; e < 4; ++e) num = mfma16(a[e], qf[c][e], num);
    }
    write(i, num / den);
  }
  }  // segments
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Bytes of one piece's slot: sums, reference maxima and row sums of its waves.
size_t slot_bytes(int d) { return (size_t)kWaves * (d / 8 + 2) * 64 * 4; }

constexpr int kPiecesPerItem = 16;

size_t items_of(int B, int H, int n_q) { return (size_t)B * H * ((n_q + kQB - 1) / kQB); }

// Workgroups the card runs at once: one per CU at d = 128 (128 KB of LDS),
// two at d = 64.
int resident(int d) { return d == 128 ? 256 : 512; }

// The most ranges a launch is cut into, and the bytes of the pieces' slots
// (two per range) and the items' arrival counters.
size_t max_ranges(int d, size_t items) { return std::min<size_t>(items * kPiecesPerItem, resident(d)); }
size_t partial_bytes(int d, size_t items, size_t ranges) {
  return ranges * 2 * slot_bytes(d) + align256(items * 4);
}

}  // namespace

size_t attention_f32_partial_bytes(int B, int H, int d, int n_q) {
  const size_t items = items_of(B, H, n_q);
  return partial_bytes(d, items, max_ranges(d, items));
}

// One whole item per workgroup, or G equal ranges of all items' steps. The
// model, in steps (64 keys of an item, 3.6 us at d = 128): rounds of resident
// workgroups, each as long as its steps plus 1.5 per segment (first loads,
// stream merge, epilogue); a cut item adds 1 plus 0.1 per piece (partials out,
// arrival, merge). Whole items in several rounds end in a tail of half the
// longest. (8 heads x d128, 1170 queries, lists of 5 and 7 pages of 392: equal
// pieces per head, two rounds of unequal ones, took 183 us.)
size_t plan_attention_f32(AttnParams& p, int B, int H, int d, int n_q, int P, const int* list_len, size_t avail) {
  const int64_t nqb = (n_q + kQB - 1) / kQB;
  const int64_t items = (int64_t)items_of(B, H, n_q), slots = resident(d);
  int64_t off[HSA_MAX_HEADS + 1], longest = 1;
  off[0] = 0;
  for (int h = 0; h < H; ++h) {
    const int64_t tiles = (int64_t)std::max(1, list_len[h]) * ((P + kTK - 1) / kTK);
    longest = std::max(longest, (tiles + 1) / 2);
    off[h + 1] = off[h] + nqb * ((tiles + 1) / 2);
  }
  int64_t T = B * off[H];
  double best = items <= slots ? longest + 1.5 : (double)T / slots + 1.5 * items / slots + 0.5 * longest;
  int64_t G = 0;  // 0: whole items
  auto consider = [&](int64_t g) {
    // (the kernel numbers steps in 32 bits)
    if (T > INT32_MAX / 2 || g > (int64_t)max_ranges(d, items) || g > T || partial_bytes(d, items, g) > avail) return;
    const double pieces = std::ceil((double)longest * g / T) + 1;
    const double cost = (double)T / g + 1.5 * (1.0 + (double)items / g) + 1.0 + 0.1 * pieces;
    if (cost < best) {
      best = cost;
      G = g;
    }
  };
  for (int j = 2; j <= kPiecesPerItem; ++j) consider(items * j);
  consider(slots);
  const bool whole = G == 0;
  if (whole) {  // every item counts as one step
    for (int h = 0; h <= H; ++h) off[h] = h * nqb;
    T = G = items;
  }
  for (int h = 0; h <= H; ++h) p.sc.sk_head_off[h] = (int32_t)off[h];
  p.sc.sk_g = (int32_t)G;
  p.sc.sk_q = (int32_t)(T / G);
  p.sc.sk_rm = (int32_t)(T % G);
  p.sc.n_chead = whole ? 0 : 1;
  p.n_ctr = whole ? 0 : (int32_t)items;
  return whole ? 0 : partial_bytes(d, items, G);
}

void set_partials_f32(AttnParams& p, int d, void* base) {
  p.part_o = static_cast<float*>(base);
  p.attn_ctr = reinterpret_cast<int32_t*>(static_cast<uint8_t*>(base) + (size_t)p.sc.sk_g * 2 * slot_bytes(d));
}

hipError_t launch_attention_f32(int d, const AttnParams& p, hipStream_t s) {
  const dim3 grid(p.sc.sk_g), block(64 * kWaves);
  if (p.blist) {
    if (d == 128) attn_f32_kernel<128, true><<<grid, block, 0, s>>>(p);
    else attn_f32_kernel<64, true><<<grid, block, 0, s>>>(p);
  } else {
    if (d == 128) attn_f32_kernel<128, false><<<grid, block, 0, s>>>(p);
    else attn_f32_kernel<64, false><<<grid, block, 0, s>>>(p);
  }
  return hipGetLastError();
}

}  // namespace hsa
