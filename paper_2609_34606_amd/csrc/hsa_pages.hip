// Page append: new keys and values of a chunk, token-major as a projection
// writes them, copied into their pool slots in the pool's layouts (key pages
// [P][d], value pages d-major [d][P]), optionally in cube order.
//
// Cube order (App. "Block Sparse Attention", the flattening index of
// (C_t, C_h, C_w) cubes): the tokens of a page of T frames x H x W are
// stored cube by cube, so that a run of B = C_t C_h C_w consecutive stored
// tokens is one spatio-temporal cube, and a key block of the head-adaptive
// sparse branch is a cube. The paper assumes that the cube divides the
// latent; at 480p a frame is 30 x 52 tokens, so H = 30 is not a multiple of
// C_h = 8 (or 4). Cubes that fit whole come first, in the paper's order
// (cube t index, then h, then w; tokens in (t, h, w) order inside a cube);
// the truncated cubes along the far edges follow in the same order. When the
// extents divide, this is exactly the paper's index.
#include <algorithm>

#include "hsa_device.h"
#include "hsa_kernels.h"

namespace hsa {
namespace {

constexpr int kTok = 64;  // tokens per workgroup

// 16 bytes at an element's alignment (one global access)
template <typename T>
struct Vec16;
template <>
struct Vec16<uint16_t> {
  typedef uint32_t type __attribute__((ext_vector_type(4), aligned(2)));
};
template <>
struct Vec16<float> {
  typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4)));
};

// One (b, new page, head, 64-token run) per workgroup: key rows copied 16
// bytes at a time, value rows transposed through LDS into 16-byte pieces of
// the d-major page rows (128 bytes of a row per workgroup in bf16). Bound: HBM
// (each page read and written once); a lane has all its loads in flight at
// once. Neighbouring workgroups take the heads of one run, whose rows are
// neighbours in the source. 3 pages of 1560 tokens, 12 heads x d128, bf16 in
// cube order (57.5 MB read and written): 11.7 us, 4.9 TB/s (a 1 GiB copy: 5.1);
// with 2-byte accesses it took 37 us.
// The LDS rows are one dword longer than d: the 8 (bf16) or 16 (fp32) token
// groups that a wave reads at once, 8 or 4 rows apart, fall on their own banks.
template <typename T, int D>
__global__ __launch_bounds__(256) void page_write_kernel(PageWriteParams p) {
  using V16 = typename Vec16<T>::type;
  constexpr int E = 16 / sizeof(T);              // elements per 16 bytes
  constexpr int CPR = D / E;                     // 16-byte chunks per token row
  constexpr int NLD = kTok * CPR / 256;          // chunks per thread and tensor
  constexpr int RW = D * (int)sizeof(T) / 4 + 1; // dwords per LDS row
  constexpr int EPW = 4 / sizeof(T);             // elements (dims) per dword
  __shared__ uint32_t vs[kTok * RW];
  const int tid = threadIdx.x;
  const int run = blockIdx.x / p.H, h = blockIdx.x % p.H;
  const int b = blockIdx.z / p.n_pages, pg = blockIdx.z % p.n_pages;
  const int i0 = run * kTok;
  const int n = min(kTok, p.P - i0);             // a multiple of 8
  const int slot = clampi(ld_const(p.page_table + (size_t)b * p.max_pages + p.first_page + pg), 0,
                          p.num_slots - 1);
  const T* ksrc = static_cast<const T*>(p.k_src);
  const T* vsrc = static_cast<const T*>(p.v_src);
  T* kdst = static_cast<T*>(p.k) + ((size_t)slot * p.H + h) * p.P * D;
  T* vdst = static_cast<T*>(p.v) + ((size_t)slot * p.H + h) * D * p.P;
  // source row of stored token i: token src_of[i] of the page in raster order
  size_t row[NLD];
#pragma unroll
  for (int l = 0; l < NLD; ++l) {
    const int i = i0 + min((tid + 256 * l) / CPR, n - 1);
    const int s = p.src_of ? clampi(p.src_of[i], 0, p.P - 1) : i;
    row[l] = (((size_t)b * p.n_pages + pg) * p.P + s) * p.H + h;
  }
  V16 k[NLD], v[NLD];
#pragma unroll
  for (int l = 0; l < NLD; ++l) v[l] = *reinterpret_cast<const V16*>(vsrc + row[l] * D + tid % CPR * E);
#pragma unroll
  for (int l = 0; l < NLD; ++l) k[l] = *reinterpret_cast<const V16*>(ksrc + row[l] * D + tid % CPR * E);
#pragma unroll
  for (int l = 0; l < NLD; ++l) {
    uint32_t* dst = vs + (tid + 256 * l) / CPR * RW + tid % CPR * 4;
#pragma unroll
    for (int w = 0; w < 4; ++w) dst[w] = v[l][w];
  }
#pragma unroll
  for (int l = 0; l < NLD; ++l) {
    const int i = (tid + 256 * l) / CPR;
    if (i < n) *reinterpret_cast<V16*>(kdst + (size_t)(i0 + i) * D + tid % CPR * E) = k[l];
  }
  __syncthreads();
  // item x: token group x % TG (16 bytes of a row), dword column x / TG
  constexpr int TG = kTok / E;
#pragma unroll
  for (int x = tid; x < TG * (RW - 1); x += 256) {
    const int t0 = x % TG * E, w = x / TG;
    if (t0 >= n) continue;
    uint32_t e[E];
#pragma unroll
    for (int t = 0; t < E; ++t) e[t] = vs[(t0 + t) * RW + w];
    T* dst = vdst + (size_t)(w * EPW) * p.P + i0 + t0;
    if constexpr (EPW == 2) {
      V16 lo, hi;  // dims 2 w and 2 w + 1
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        lo[t] = (e[2 * t] & 0xffffu) | (e[2 * t + 1] << 16);
        hi[t] = (e[2 * t] >> 16) | (e[2 * t + 1] & 0xffff0000u);
      }
      *reinterpret_cast<V16*>(dst) = lo;
      *reinterpret_cast<V16*>(dst + p.P) = hi;
    } else {
      *reinterpret_cast<V16*>(dst) = V16{e[0], e[1], e[2], e[3]};
    }
  }
}

}  // namespace

hipError_t launch_page_write(int dtype, int d, int B, const PageWriteParams& p, hipStream_t s) {
  const dim3 grid((p.P + kTok - 1) / kTok * p.H, 1, B * p.n_pages);
  if (dtype == HSA_DTYPE_BF16) {
    if (d == 128) page_write_kernel<uint16_t, 128><<<grid, 256, 0, s>>>(p);
    else page_write_kernel<uint16_t, 64><<<grid, 256, 0, s>>>(p);
  } else {
    if (d == 128) page_write_kernel<float, 128><<<grid, 256, 0, s>>>(p);
    else page_write_kernel<float, 64><<<grid, 256, 0, s>>>(p);
  }
  return hipGetLastError();
}

int cube_order(int T, int H, int W, int ct, int ch, int cw, int32_t* src_of) {
  const int Nt = T / ct, Nh = H / ch, Nw = W / cw;                    // whole cubes
  const int Mt = (T + ct - 1) / ct, Mh = (H + ch - 1) / ch, Mw = (W + cw - 1) / cw;
  int n = 0;
  auto emit_cube = [&](int a, int bh, int c) {
    for (int t = a * ct; t < std::min(T, (a + 1) * ct); ++t)
      for (int hh = bh * ch; hh < std::min(H, (bh + 1) * ch); ++hh)
        for (int w = c * cw; w < std::min(W, (c + 1) * cw); ++w) src_of[n++] = (t * H + hh) * W + w;
  };
  for (int a = 0; a < Nt; ++a)
    for (int bh = 0; bh < Nh; ++bh)
      for (int c = 0; c < Nw; ++c) emit_cube(a, bh, c);
  const int whole = n;
  for (int a = 0; a < Mt; ++a)
    for (int bh = 0; bh < Mh; ++bh)
      for (int c = 0; c < Mw; ++c)
        if (a >= Nt || bh >= Nh || c >= Nw) emit_cube(a, bh, c);
  return whole;
}

}  // namespace hsa
