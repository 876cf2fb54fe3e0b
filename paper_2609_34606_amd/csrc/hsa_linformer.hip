// Linformer compression of pages (Sec. 3.3 "Linear branch"; App. "Linear
// Branch"): with one page as the projection segment (L = P), every page of
// every head is compressed once, when it is written,
//   ck = E_K^T K   (r x d),     cv = (E_V^T V)^T   (d x r, stored d-major),
// with the head's projections given as e_k[h][j][t] = E_K^(h)[t][j]. The
// compressed pages form a KV pool of page size r that the attention kernels
// read like any other pool.
//
// bf16: both products contract over the page's tokens, and neither needs the
// other's operands, so a work item is one product of one (page part, head):
// 64-token tiles of the projection (rank-major rows) and of the data (value
// rows as stored; key rows transposed to [d][token] on the way into LDS),
// 32x32x16 bf16 MFMAs with fp32 accumulation. A page is split into parts only
// when there are too few (page, head) pairs to fill the chip; parts write fp32
// partials that a second kernel sums in order.
//
// Bound: HBM (the pages; the projections come from L2). Under load a tile
// takes about 5 us to arrive, so what counts is the bytes in flight per CU:
// the data of the next two tiles is in registers or on its way while a tile is
// computed, at four workgroups per CU. Measured, 12 heads x d128, rank 64, pages
// of 1560 tokens: 48 pages (460 MB) 118 us, 3.9 TB/s counting each page once,
// and 123 pages 284 us, 4.1 TB/s; one workgroup per page and head with both
// products, loading a tile and then computing it, took 157 and 288 us, the same
// with one tile prefetched 132 us for the 48. Five workgroups per CU spill
// registers: 140 us.
#include <type_traits>

#include "hsa_device.h"
#include "hsa_kernels.h"

namespace hsa {
namespace {

constexpr int kT = 64;          // tokens per LDS tile
constexpr int kRow = kT * 2;    // bytes per LDS row: 64 bf16 tokens

// 16-byte chunk swizzle of 128-byte LDS rows: 16 consecutive rows read at one
// logical chunk land on distinct bank groups.
__device__ __forceinline__ int swz(int row) { return ((row >> 1) ^ (row >> 4)) & 7; }

// Four outputs in one 8-byte store at an element's alignment: nothing more is
// asked of ck and cv.
typedef uint32_t u32x2e __attribute__((ext_vector_type(2), aligned(2)));

template <int D, int R>
struct CompressSmem {
  uint8_t x[D * kRow];     // K^T or V tile [d][64 tokens]
  uint8_t e[2][R * kRow];  // E_K^T or E_V^T tiles [j][64 tokens]
};

template <int D, int R, bool kSmallP>
__global__ __launch_bounds__(256, R * D <= 64 * 128 ? 4 : 3) void compress_bf16_kernel(CompressParams p) {
  constexpr int DQ = D / 4, KG = 256 / DQ, KPT = kT / KG;  // key loads: 4 dims x KPT tokens
  constexpr int NV = D / 32;           // 16-byte value loads per thread (8 rows per wave each)
  constexpr int NE = R / 32;           // 16-byte projection loads per thread
  // 32x32 output tiles, projection rows by d columns: waves in a WM x WN grid
  // of NA x NB tiles each (rank 32 at d = 64 leaves two waves without one)
  constexpr int NMD = D / 32, NMR = R / 32;
  constexpr int WM = NMR > 1 ? 2 : 1, WN = 4 / WM < NMD ? 4 / WM : NMD;
  constexpr int NA = NMR / WM, NB = NMD / WN;
  static_assert(KPT == 2 * NV, "key and value tiles take the same registers");
  __shared__ __attribute__((aligned(16))) CompressSmem<D, R> sm;

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroup ids go round-robin to the 8 XCDs. Each XCD takes consecutive items
  // (head, page, part) of the key product and then as many of the value
  // product, so that the few projections it reads stay in its L2 and every XCD
  // has the same work: a value tile, whose rows are 128-byte pieces, takes a
  // sixth longer than a key tile. (head, product, page, part) gave XCDs two heads
  // of one product and one of the other at 12 heads: 123 pages 304 us, now 284;
  // 288 with both products in one workgroup.
  const int per = p.n_pages * p.parts, G = per * 2 * p.H;
  const int lin = (int)(blockIdx.y * gridDim.x + blockIdx.x), xcd = lin & 7;
  auto start = [&](int x) { return x * (G >> 3) + min(x, G & 7); };
  const int s0 = start(xcd), s1 = start(xcd + 1), j = lin >> 3;
  const int k0 = (s0 + 1) >> 1, v0 = s0 >> 1, nk = ((s1 + 1) >> 1) - k0;
  const bool is_k = j < nk;
  const int item = is_k ? k0 + j : v0 + (j - nk);
  const int h = item / per, pi = item % per / p.parts, part = item % p.parts, b = blockIdx.z;
  const int page = p.first_page + pi;
  const int slot = clampi(p.page_table[(size_t)b * p.max_pages + page], 0, p.num_slots - 1);
  const size_t hb = (size_t)slot * p.H + h;
  const int P = p.P;
  const int t_beg = part * p.part_len, t_end = min(P, t_beg + p.part_len);

  // ---- tile loads: one scalar base per tensor plus per-lane offsets, fixed
  // for the whole page. Rows of 64 tokens (values, projections): instruction n
  // of a wave covers 8 rows, source chunk (lane % 8) ^ swz(r) of row r lands at
  // chunk lane % 8. Keys: 4 dims x KPT tokens per thread.
  const uint16_t* xb = static_cast<const uint16_t*>(is_k ? p.k : p.v) + hb * P * D;      // [P][D] or [D][P]
  const uint16_t* eb = static_cast<const uint16_t*>(is_k ? p.e_k : p.e_v) + (size_t)h * R * P;  // [R][P]
  const int dq = tid % DQ, kg = tid / DQ;
  auto row_of = [&](int n_inst, int n) { return (wave * n_inst + n) * 8 + (lane >> 3); };
  auto col_of = [&](int r) { return 8 * ((lane & 7) ^ swz(r)); };
  auto row_off = [&](int n_inst, int n) {
    const int r = row_of(n_inst, n);
    return (uint32_t)(r * P + (kSmallP ? min(col_of(r), P - 8) : col_of(r))) * 2u;
  };
  uint32_t v_off[NV], e_off[NE];
#pragma unroll
  for (int n = 0; n < NV; ++n) v_off[n] = row_off(NV, n);
#pragma unroll
  for (int n = 0; n < NE; ++n) e_off[n] = row_off(NE, n);
  const uint32_t k_off = (uint32_t)(kg * KPT * D + dq * 4) * 2u;
  // A lane's operand of 16-token step ks in row block n (32 rows) of a tile
  // sits at (o ^ 32 (ks ^ n)) + n blocks: swz of a row 32 n further differs by
  // 2 n, and chunks are 16 bytes.
  const int mt0 = (wave % WM) * NA, nt0 = (wave / WM) * NB;
  const bool active = wave / WM < WN;
  const uint32_t oa = (uint32_t)((mt0 * 32 + l32) * kRow + ((half ^ swz(mt0 * 32 + l32)) << 4));
  const uint32_t ob = (uint32_t)((nt0 * 32 + l32) * kRow + ((half ^ swz(nt0 * 32 + l32)) << 4));
  // The walk, for keys (kind true) or values: each compiled by itself, which
  // takes fewer registers than one walk with both loads.
  f32x16 acc[NA][NB];
#pragma unroll
  for (int m = 0; m < NA; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) acc[m][n] = f32x16{0};
  auto walk = [&](auto kind) {
  constexpr bool K = decltype(kind)::value;
  u32x4 x[2][NV];           // data of two tiles
  // tile at t0: the 64-token window ending at the page end when fewer tokens
  // remain, or the whole page when it is shorter than a tile (clamped)
  auto window = [&](int t0) { return kSmallP ? 0 : min(t0, P - kT); };
  auto load_x = [&](int t0, u32x4 (&xr)[NV]) {
    if constexpr (K) {
      const char* src = reinterpret_cast<const char*>(xb + (size_t)window(t0) * D);
      u32x2 kr[KPT];
#pragma unroll
      for (int e = 0; e < KPT; ++e) {
        uint32_t off = k_off + e * D * 2;
        if constexpr (kSmallP) off -= (uint32_t)(max(0, kg * KPT + e - (P - 1)) * D * 2);
        kr[e] = *reinterpret_cast<const u32x2*>(src + off);
      }
#pragma unroll
      for (int n = 0; n < NV; ++n) xr[n] = u32x4{kr[2 * n].x, kr[2 * n].y, kr[2 * n + 1].x, kr[2 * n + 1].y};
    } else {
      const char* src = reinterpret_cast<const char*>(xb + window(t0));
#pragma unroll
      for (int n = 0; n < NV; ++n) xr[n] = ld_global16(src + v_off[n]);
    }
  };
  // projections go straight into LDS, issued before the same step's data
  // loads: waiting for them leaves those in flight
  auto load_e = [&](int t0, int buf) {
    const char* src = reinterpret_cast<const char*>(eb + window(t0));
#pragma unroll
    for (int n = 0; n < NE; ++n) g2lds16_hidden(src + e_off[n], sm.e[buf] + (wave * NE + n) * 1024);
  };

  // one tile: registers -> LDS, the loads of the tile after next, products.
  // kPair: the loads of the next two tiles after the second of two; the two
  // 128-byte pieces of a value row, which share a cache line, then meet in the
  // cache. d = 64, rank 64, 16 heads, 96 pages of 1560: 175 -> 169 us; at d =
  // 128, where a tile is twice as long, 24 pages took 47.5 -> 48.8 us.
  constexpr bool kPair = !K && D == 64;
  constexpr int kLoadsX = K ? KPT : NV;
  auto step = [&](int t0, auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    u32x4 (&xr)[NV] = x[buf];
    // valid tokens of this tile's window: [lo, hi), multiples of 8; the others
    // are zeros in one operand (keys; the projection of the values)
    const int lo = t0 - window(t0), hi = lo + min(kT, t_end - t0);
    if constexpr (K) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int d = dq * 4 + c;
        uint32_t w[KPT / 2];
#pragma unroll
        for (int e = 0; e < KPT / 2; ++e) {
          const uint32_t x0 = c < 2 ? xr[e].x : xr[e].y, x1 = c < 2 ? xr[e].z : xr[e].w;
          w[e] = (c & 1) ? __builtin_amdgcn_perm(x1, x0, 0x07060302) : __builtin_amdgcn_perm(x1, x0, 0x05040100);
        }
        const int key0 = kg * KPT;  // KPT (4 or 8) tokens, on one side of lo and hi
        if (key0 < lo || key0 >= hi)
#pragma unroll
          for (int e = 0; e < KPT / 2; ++e) w[e] = 0;
        uint8_t* dst = &sm.x[d * kRow + (((key0 >> 3) ^ swz(d)) << 4) + (key0 & 7) * 2];
        if constexpr (KPT == 8) *reinterpret_cast<u32x4*>(dst) = u32x4{w[0], w[1], w[2], w[3]};
        else *reinterpret_cast<u32x2*>(dst) = u32x2{w[0], w[1]};
      }
    } else {
#pragma unroll
      for (int n = 0; n < NV; ++n) *reinterpret_cast<u32x4*>(sm.x + ((wave * NV + n) * 64 + lane) * 16) = xr[n];
    }
    // this tile's projection has landed: only the next tile's data is later
    if ((!kPair || buf == 0) && t0 + kT < t_end) wait_vmcnt<kLoadsX>();
    else wait_vmcnt<0>();
    if constexpr (!K) {
      if (lo > 0 || hi < kT) {  // each lane clears what it loaded
#pragma unroll
        for (int n = 0; n < NE; ++n) {
          const int col = col_of(row_of(NE, n));
          if (col < lo || col >= hi)
            *reinterpret_cast<u32x4*>(sm.e[buf] + ((wave * NE + n) * 64 + lane) * 16) = u32x4{0};
        }
      }
    }
    lds_barrier();
    if (t0 + kT < t_end) load_e(t0 + kT, buf ^ 1);
    if constexpr (!kPair) {
      if (t0 + 2 * kT < t_end) load_x(t0 + 2 * kT, xr);
    } else if constexpr (buf == 1) {
      if (t0 + kT < t_end) load_x(t0 + kT, x[0]);
      if (t0 + 2 * kT < t_end) load_x(t0 + 2 * kT, x[1]);
    }
    if (active) {
      // (opaque, so that the eight operand offsets are recomputed per tile
      // instead of held across the walk)
      uint32_t o_a = oa, o_b = ob;
      asm volatile("" : "+v"(o_a), "+v"(o_b));
#pragma unroll
      for (int ks = 0; ks < kT / 16; ++ks) {
        u32x4 a[NA];
#pragma unroll
        for (int m = 0; m < NA; ++m) a[m] = ld_lds16(sm.e[buf] + (o_a ^ ((ks ^ m) << 5)) + m * 32 * kRow);
#pragma unroll
        for (int n = 0; n < NB; ++n) {
          const u32x4 bb = ld_lds16(sm.x + (o_b ^ ((ks ^ n) << 5)) + n * 32 * kRow);
#pragma unroll
          for (int m = 0; m < NA; ++m) acc[m][n] = mfma32(a[m], bb, acc[m][n]);
        }
      }
    }
    lds_barrier();
  };
  if (t_beg < t_end) {
    load_e(t_beg, 0);
    load_x(t_beg, x[0]);
    if (t_beg + kT < t_end) load_x(t_beg + kT, x[1]);
  }
  for (int t0 = t_beg; t0 < t_end; t0 += 2 * kT) {
    step(t0, std::integral_constant<int, 0>{});
    if (t0 + kT < t_end) step(t0 + kT, std::integral_constant<int, 1>{});
  }
  };
  if (is_k) walk(std::true_type{});
  else walk(std::false_type{});

  // lane holds column d = 32 nt + lane % 32 of each tile, projection rows
  // 32 mt + 8 (r / 4) + 4 (lane / 32) + r % 4
  if (!active) return;
  uint16_t* ck = static_cast<uint16_t*>(p.ck) + hb * R * D;   // [R][D]
  uint16_t* cv = static_cast<uint16_t*>(p.cv) + hb * D * R;   // [D][R]
  float* part_out = p.parts > 1
      ? p.partial + ((((size_t)b * p.H + h) * p.n_pages + pi) * p.parts + part) * (2 * R * D)
      : nullptr;
#pragma unroll
  for (int m = 0; m < NA; ++m)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int d = 32 * (nt0 + n) + l32;
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        const int j = 32 * (mt0 + m) + 8 * r4 + 4 * half;
        const f32x4 v = f32x4{acc[m][n][4 * r4], acc[m][n][4 * r4 + 1], acc[m][n][4 * r4 + 2], acc[m][n][4 * r4 + 3]};
        if (is_k) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (part_out) part_out[(j + r) * D + d] = v[r];
            else ck[(j + r) * D + d] = (uint16_t)(pack_bf16(v[r], 0.f) & 0xffffu);
          }
        } else if (part_out) {
          *reinterpret_cast<f32x4*>(part_out + R * D + d * R + j) = v;
        } else {
          *reinterpret_cast<u32x2e*>(cv + d * R + j) = u32x2e{pack_bf16(v.x, v.y), pack_bf16(v.z, v.w)};
        }
      }
    }
}

// Sum of a page's parts in part order, rounded once to bf16. One workgroup
// per (1024 outputs, page, head), four consecutive outputs per thread.
constexpr int kReduceChunk = 1024;

__global__ __launch_bounds__(256) void compress_reduce_kernel(CompressParams p) {
  const int RD = p.R * p.D;
  const int chunks = 2 * RD / kReduceChunk;
  const int pi = blockIdx.x / chunks, c = blockIdx.x % chunks, h = blockIdx.y, b = blockIdx.z;
  const int page = p.first_page + pi;
  const int slot = clampi(p.page_table[(size_t)b * p.max_pages + page], 0, p.num_slots - 1);
  const size_t hb = (size_t)slot * p.H + h;
  const float* src = p.partial + (((size_t)b * p.H + h) * p.n_pages + pi) * p.parts * (2 * RD);
  const int e = c * kReduceChunk + 4 * threadIdx.x;
  f32x4 s = *reinterpret_cast<const f32x4*>(src + e);
  for (int k = 1; k < p.parts; ++k) s += *reinterpret_cast<const f32x4*>(src + (size_t)k * 2 * RD + e);
  uint16_t* dst = (e < RD ? static_cast<uint16_t*>(p.ck) + hb * RD + e
                          : static_cast<uint16_t*>(p.cv) + hb * RD + (e - RD));
  *reinterpret_cast<u32x2e*>(dst) = u32x2e{pack_bf16(s.x, s.y), pack_bf16(s.z, s.w)};
}

// fp32 inputs: plain VALU products, fp32 accumulation in token order (small
// shapes; fp32 end to end).
__global__ __launch_bounds__(256) void compress_f32_kernel(CompressParams p) {
  const int pi = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int page = p.first_page + pi;
  const int slot = clampi(p.page_table[(size_t)b * p.max_pages + page], 0, p.num_slots - 1);
  const size_t hb = (size_t)slot * p.H + h;
  const int P = p.P, R = p.R, D = p.D;
  const float* kb = static_cast<const float*>(p.k) + hb * P * D;
  const float* vb = static_cast<const float*>(p.v) + hb * D * P;
  const float* ekb = static_cast<const float*>(p.e_k) + (size_t)h * R * P;
  const float* evb = static_cast<const float*>(p.e_v) + (size_t)h * R * P;
  float* ck = static_cast<float*>(p.ck) + hb * R * D;
  float* cv = static_cast<float*>(p.cv) + hb * D * R;
  for (int e = threadIdx.x; e < 2 * R * D; e += 256) {
    float s = 0.f;
    if (e < R * D) {
      const int j = e / D, d = e % D;
      for (int t = 0; t < P; ++t) s = fmaf(ekb[(size_t)j * P + t], kb[(size_t)t * D + d], s);
      ck[e] = s;
    } else {
      const int d = (e - R * D) / R, j = (e - R * D) % R;
      for (int t = 0; t < P; ++t) s = fmaf(vb[(size_t)d * P + t], evb[(size_t)j * P + t], s);
      cv[e - R * D] = s;
    }
  }
}

template <int D, int R>
void launch_compress_bf16(const CompressParams& p, int B, hipStream_t s) {
  const dim3 grid(p.n_pages * p.parts, 2 * p.H, B);
  if (p.P < kT) compress_bf16_kernel<D, R, true><<<grid, 256, 0, s>>>(p);
  else compress_bf16_kernel<D, R, false><<<grid, 256, 0, s>>>(p);
}

}  // namespace

hipError_t launch_compress(int dtype, int B, const CompressParams& p, hipStream_t s) {
  if (dtype != HSA_DTYPE_BF16) {
    compress_f32_kernel<<<dim3(p.n_pages, p.H, B), 256, 0, s>>>(p);
    return hipGetLastError();
  }
  if (p.D == 128) {
    if (p.R == 32) launch_compress_bf16<128, 32>(p, B, s);
    else if (p.R == 64) launch_compress_bf16<128, 64>(p, B, s);
    else launch_compress_bf16<128, 128>(p, B, s);
  } else {
    if (p.R == 32) launch_compress_bf16<64, 32>(p, B, s);
    else if (p.R == 64) launch_compress_bf16<64, 64>(p, B, s);
    else launch_compress_bf16<64, 128>(p, B, s);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.parts == 1) return e;
  // 2 R d is a multiple of kReduceChunk for every supported (R, d)
  compress_reduce_kernel<<<dim3(p.n_pages * (2 * p.R * p.D / kReduceChunk), p.H, B), 256, 0, s>>>(p);
  return hipGetLastError();
}

}  // namespace hsa
