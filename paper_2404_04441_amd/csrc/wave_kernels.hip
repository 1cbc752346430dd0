// gfx950 kernels of libwave other than the step kernel (whose templates
// live in step_kernels.h): the CPML boundary passes, setup, decode,
// gather/scatter, gradient and fill kernels, and the launchers.
#include "step_kernels.h"

namespace wave {
namespace {

// n / d for n < 2^31: (n + mulhi(n, m)) >> s.
struct FastDiv {
  unsigned d, m, s;
  explicit FastDiv(unsigned div = 1) : d(div), s(0) {
    while ((1ull << s) < d) ++s;
    m = static_cast<unsigned>((((1ull << s) - d) << 32) / d + 1);
  }
  __device__ unsigned operator()(unsigned n) const { return (__umulhi(n, m) + n) >> s; }
};

// ------------------------------------------------------------ CPML boundary
//
// The convolutional PML the paper names as its boundary (Sec. II, Sec.
// IV-A), for the second-order acoustic equation: per axis a memory variable
// psi_a of the first derivative and zeta_a of the second,
//   psi_a^n  = b psi_a^{n-1}  + a D1_a p^n
//   zeta_a^n = b zeta_a^{n-1} + a (D2_a p^n + D1_a psi_a^n)
//   p^{n+1}  = (plain leapfrog step) + m sum_a (D1_a psi_a^n + zeta_a^n).
// The psi update runs before the step, along y and z by rows of the boundary
// shell and along x over its slabs.  The correction runs after it: by rows for the
// y and z terms where the step applies the x part itself, else a thread per node of
// the shell for all three.

// Node t of the boundary shell for layers of E nodes: the planes of the z
// layers, then in the remaining planes the rows of the y layers, then in the
// remaining rows the columns of the x layers (every shell node once).  32-bit
// index arithmetic: the host keeps the shell below 2^31 nodes.
struct Shell {
  unsigned nx, ny, nz, E, cz, cy, cx, mz, my, n0, n1, n2;
  __host__ __device__ Shell(int e, int x, int y, int z) {
    nx = x;
    ny = y;
    nz = z;
    E = e;
    cz = nz < 2u * E ? nz : 2u * E;
    cy = ny < 2u * E ? ny : 2u * E;
    cx = nx < 2u * E ? nx : 2u * E;
    mz = nz - cz;
    my = ny - cy;
    n0 = cz * ny * nx;
    n1 = mz * cy * nx;
    n2 = mz * my * cx;
  }
  __host__ __device__ unsigned count() const { return n0 + n1 + n2; }
  // the k-th layer plane and y-layer row
  __device__ unsigned z_at(unsigned k) const { return k < E ? k : nz - cz + k; }
  __device__ unsigned y_at(unsigned k) const { return k < E ? k : ny - cy + k; }
  __device__ void node(unsigned t, int &x, int &y, int &z) const {
    if (t < n0) {
      const unsigned k = t / (ny * nx), r = t - k * (ny * nx);
      z = static_cast<int>(k < E ? k : nz - cz + k);
      y = static_cast<int>(r / nx);
      x = static_cast<int>(r - (r / nx) * nx);
      return;
    }
    t -= n0;
    if (t < n1) {
      const unsigned row = t / nx, k = row % cy;
      z = static_cast<int>(E + row / cy);
      y = static_cast<int>(k < E ? k : ny - cy + k);
      x = static_cast<int>(t - row * nx);
      return;
    }
    t -= n1;
    const unsigned row = t / cx, k = t - row * cx;
    z = static_cast<int>(E + row / my);
    y = static_cast<int>(E + row % my);
    x = static_cast<int>(k < E ? k : nx - cx + k);
  }
};

// Per-axis addressing of one node: coordinate i along the axis, axis length
// n, field stride, and the node's offset in the axis' slab array without its
// slab index (plus the slab stride), 32-bit.
struct AxisAt {
  int i, n;
  unsigned stride, slab_rest, slab_stride;
};

__device__ __forceinline__ AxisAt axis_at(const CpmlArgs &c, int a, int x, int y, int z) {
  const unsigned nx = c.nx, ny = c.ny, W2 = 2u * c.W;
  AxisAt r;
  if (a == 0) {
    r = {x, c.nx, 1u, (static_cast<unsigned>(z) * ny + y) * W2, 1u};
  } else if (a == 1) {
    r = {y, c.ny, nx, static_cast<unsigned>(z) * W2 * nx + x, nx};
  } else {
    r = {z, c.nz, nx * ny, static_cast<unsigned>(y) * nx + x, ny * nx};
  }
  return r;
}

// psi_a at the node k steps along the axis (zero outside the layers).
__device__ __forceinline__ float psi_k(const CpmlArgs &c, int a, const AxisAt &A, int k) {
  const int s = slab_index(A.i + k, A.n, c.W);
  return s < 0 ? 0.f : c.psi[a][A.slab_rest + static_cast<unsigned>(s) * A.slab_stride];
}

// cur at the node k steps along the axis (zero outside the grid).
__device__ __forceinline__ float cur_k(const float *cur, unsigned o, const AxisAt &A, int k) {
  const int j = A.i + k;
  return (j < 0 || j >= A.n) ? 0.f : cur[static_cast<int>(o) + k * static_cast<int>(A.stride)];
}

// A lane's kRowNodes nodes of a row: kRowNodes / VEC vectors of VEC nodes, 64
// vectors apart (whole rows need nx % VEC == 0; narrower vectors, more of
// them).
constexpr int kRowNodes = 4;
template <int VEC> struct Row {
  Words<VEC * 4> v[kRowNodes / VEC];
  __device__ float at(int e) const { return __uint_as_float(v[e / VEC].w[e % VEC]); }
};
template <int VEC> __device__ __forceinline__ Row<VEC> ld_row(rsrc_t r, uint32_t xo) {
  Row<VEC> out;
#pragma unroll
  for (int k = 0; k < kRowNodes / VEC; ++k) out.v[k] = ld_words<VEC * 4, 0>(r, xo + k * (256u * VEC), 0u);
  return out;
}
template <int VEC> __device__ __forceinline__ void st_row(const float *v, rsrc_t r, uint32_t xo) {
#pragma unroll
  for (int k = 0; k < kRowNodes / VEC; ++k)
    st_words<VEC * 4, 0>(row_put<kF32, VEC>(v + k * VEC), r, xo + k * (256u * VEC), 0u);
}

// The row kernels' order of work.  A wavefront owns 256 consecutive nodes
// of one row of the shell, so that the row, its layers and its neighbour rows
// are scalars: one resource per neighbour row, without records where the row
// lies outside (its loads return zero), and no address or mask arithmetic per
// lane.  With a thread per vector of the whole shell these kernels were bound
// by that arithmetic, five integer divisions per thread among it.  A row's
// neighbours along z (z layers) or y (y layers) are other rows of the shell:
// each XCD, with an L2 of its own, takes a contiguous run of rows (hardware
// dispatches workgroups round-robin over the 8 XCDs), and the z-layer planes
// are visited in bundles of kBundle rows, all planes of a bundle and then the
// next bundle, so that the rows in flight on an XCD hold whole z lines.
// Every XCD takes an eighth of each part (z-layer rows, y-layer rows, nodes of
// the x slabs), so that they end together.  Measured at 512^3, W = 20: the psi
// update (before: a row kernel of 95 us and a column kernel of 37 us) 83 us,
// 0.44 GB; the correction reads 0.45 instead of 0.80 GB (0.50 with four rows a wavefront); at 401x333x301, where a lane held one node, a whole step went from
// 398 to 362 us.  Bundles of 4, 32 and 64 rows differ by 1%.
constexpr unsigned kBundle = 32;

struct ShellWork {
  Shell S;
  unsigned per0, per1, per2;  // workgroups (4 wavefronts) of each part per XCD
  unsigned rows0, rows1;      // rows of the first two parts
  unsigned nslab;             // vectors of the x slabs
  unsigned group;             // rows of a wavefront: consecutive planes (part 0) or rows (part 1)
  unsigned first = 0;         // this launch's first workgroup of each XCD's run
  FastDiv seg, bundle, last, cy, w2v;  // wavefronts per row; rows per bundle and in the last one; rows per y-layer plane; vectors per x-slab row
  ShellWork(const CpmlArgs &c, int E, int vx, unsigned g = 1) : S(E, c.nx, c.ny, c.nz), group(g) {
    const unsigned gz = (S.cz + g - 1) / g, gy = (S.cy + g - 1) / g;
    const unsigned nseg = (static_cast<unsigned>(c.nx) + 64 * kRowNodes - 1) / (64 * kRowNodes);
    seg = FastDiv(nseg);
    bundle = FastDiv(gz * kBundle);
    const unsigned tail = S.ny % kBundle;
    last = FastDiv(tail ? tail : kBundle);
    cy = FastDiv(gy);
    rows0 = gz * S.ny;
    rows1 = S.mz * gy;
    w2v = FastDiv(vx ? 2u * c.W / vx : 1u);
    nslab = vx ? static_cast<unsigned>(c.nz) * c.ny * (2u * c.W / vx) : 0u;
    auto share = [](size_t waves) { return static_cast<unsigned>((waves + 31) / 32); };  // 4 wavefronts, 8 XCDs
    per0 = share(size_t(rows0) * nseg);
    per1 = share(size_t(rows1) * nseg);
    per2 = share((size_t(nslab) + 63) / 64);
  }
  // launch(grid, work) until every workgroup had its turn: one launch but for
  // grids of tens of millions of rows, as a launch holds fewer than 2^32 threads
  template <typename F> void run(F &&launch) {
    constexpr unsigned kMost = 1u << 20;  // per XCD: 2^31 threads a launch
    const unsigned n = per0 + per1 + per2;
    for (first = 0; first < n; first += kMost) launch(dim3(8 * (n - first < kMost ? n - first : kMost)), *this);
  }
};

// This wavefront's part, its index there and, in the row parts, its row: part
// 0 (the rows of the z-layer planes, by bundles) or 1 (the y-layer rows of the
// remaining planes), the segment of the row; part 3 past the end.  Scalars,
// said so to the compiler: a resource it takes for divergent costs a loop
// over the lanes at each load.
struct ShellAt {
  unsigned part, wave, seg;
  unsigned k;  // the (first) row's index among the layers' planes (part 0) or rows (part 1)
  int y, z;
};

__device__ __forceinline__ ShellAt shell_at(const ShellWork &P) {
  const Shell &S = P.S;
  const unsigned xcd = blockIdx.x & 7u, j = P.first + (blockIdx.x >> 3);
  const unsigned w = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6));
  ShellAt at{};
  unsigned y = 0, z = 0, k = 0;
  if (j < P.per0) {
    at.wave = (xcd * P.per0 + j) * 4u + w;
    const unsigned r = P.seg(at.wave);
    at.seg = at.wave - r * P.seg.d;
    const unsigned b = P.bundle(r), rem = r - b * P.bundle.d;
    const bool whole = S.ny - b * kBundle >= kBundle;
    const unsigned g = whole ? rem / kBundle : P.last(rem);
    y = b * kBundle + (rem - g * (whole ? kBundle : P.last.d));
    k = g * P.group;
    z = S.z_at(k);
    at.part = r < P.rows0 ? 0u : 3u;
  } else if (j < P.per0 + P.per1) {
    at.wave = (xcd * P.per1 + j - P.per0) * 4u + w;
    const unsigned r = P.seg(at.wave);
    at.seg = at.wave - r * P.seg.d;
    const unsigned zi = P.cy(r);
    k = (r - zi * P.cy.d) * P.group;
    y = S.y_at(k);
    z = S.E + zi;
    at.part = r < P.rows1 ? 1u : 3u;
  } else {
    at.wave = (xcd * P.per2 + j - P.per0 - P.per1) * 4u + w;
    at.part = 2u;
  }
  at.part = __builtin_amdgcn_readfirstlane(at.part);
  at.seg = __builtin_amdgcn_readfirstlane(at.seg);
  at.k = __builtin_amdgcn_readfirstlane(k);
  at.y = __builtin_amdgcn_readfirstlane(static_cast<int>(y));
  at.z = __builtin_amdgcn_readfirstlane(static_cast<int>(z));
  return at;
}

// The row of nx floats at p, or nothing (every load from it is zero).
__device__ __forceinline__ rsrc_t row_at(const float *p, bool in, unsigned nx) {
  return make_rsrc(p, in ? nx * 4u : 0u);
}

template <int VEC> __device__ __forceinline__ void vload(const float *p, float *v) { lds_get<VEC>(p, v); }
template <int VEC> __device__ __forceinline__ void vstore(float *p, const float *v) { lds_put<VEC>(p, v); }

// psi_x over vector t of the x slabs (VX consecutive nodes; W and nx
// divisible by VX): contiguous in the slab array, the window of A^n in
// vectors of VX.
template <int VX>
__device__ __forceinline__ void psi_x_update(const CpmlArgs &c, const ShellWork &P, const float *__restrict__ cur,
                                             unsigned t) {
  if (t >= P.nslab) return;
  const unsigned row = P.w2v(t);  // row z ny + y of the grid
  const int s = static_cast<int>(t - row * P.w2v.d) * VX, nx = c.nx;
  const int x = s < c.W ? s : nx - 2 * c.W + s;
  const float *u = cur + static_cast<size_t>(row) * static_cast<unsigned>(nx);
  constexpr int NV = (VX + 2 * R + VX - 1) / VX;  // vectors of the window x-R .. x+VX+R-1
  float win[NV * VX];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int xk = x - R + k * VX;
#pragma unroll
    for (int e = 0; e < VX; ++e) win[k * VX + e] = 0.f;
    if (xk >= 0 && xk < nx) vload<VX>(u + xk, win + k * VX);
  }
  float *ps = c.psi[0] + static_cast<size_t>(t) * VX;
  float pv[VX];
  vload<VX>(ps, pv);
#pragma unroll
  for (int e = 0; e < VX; ++e) {
    float d = 0.f;
#pragma unroll
    for (int m = 1; m <= R; ++m) d = fmaf(c.d1w[0][m - 1], win[R + e + m] - win[R + e - m], d);
    pv[e] = fmaf(c.cb[0][x + e], pv[e], c.ca[0][x + e] * d);
  }
  vstore<VX>(ps, pv);
}

// psi_a update over the W-node layers: along y and z by rows (VEC consecutive
// x nodes per lane, nx % VEC == 0), along x over the slabs.
template <int VEC, int VX>
__global__ void __launch_bounds__(256) cpml_psi_kernel(CpmlArgs c, ShellWork P, const float *__restrict__ cur) {
  const ShellAt at = shell_at(P);
  const unsigned lane = threadIdx.x & 63u, seg = at.seg;
  const int y = at.y, z = at.z;
  if (at.part == 2) psi_x_update<VX>(c, P, cur, at.wave * 64u + lane);
  if (at.part >= 2) return;
  const unsigned nx = c.nx, ny = c.ny, W2 = 2u * c.W;
  const uint32_t xo = seg * (64u * kRowNodes * 4u) + lane * (VEC * 4u);  // past the row's end: loads zero, stores nothing
  const float *row = cur + (static_cast<size_t>(z) * ny + static_cast<unsigned>(y)) * nx;
#pragma unroll
  for (int a = 1; a < 3; ++a) {
    const int i = a == 1 ? y : z, n = a == 1 ? c.ny : c.nz;
    const int s = slab_index(i, n, c.W);
    if (s < 0) continue;
    const size_t stride = a == 1 ? nx : static_cast<size_t>(nx) * ny;
    Row<VEC> up[R], dn[R];
#pragma unroll
    for (int m = 1; m <= R; ++m) {
      up[m - 1] = ld_row<VEC>(row_at(row + m * stride, i + m < n, nx), xo);
      dn[m - 1] = ld_row<VEC>(row_at(row - m * stride, i - m >= 0, nx), xo);
    }
    const rsrc_t rp = row_at(c.psi[a] + (a == 1 ? static_cast<size_t>(z) * W2 + s : static_cast<size_t>(s) * ny + y) * nx,
                             true, nx);
    const Row<VEC> pv = ld_row<VEC>(rp, xo);
    const float ca = c.ca[a][i], cb = c.cb[a][i];
    float out[kRowNodes];
#pragma unroll
    for (int e = 0; e < kRowNodes; ++e) {
      float d = 0.f;
#pragma unroll
      for (int m = 1; m <= R; ++m)
        d = fmaf(c.d1w[a][m - 1], up[m - 1].at(e) - dn[m - 1].at(e), d);
      out[e] = fmaf(cb, pv.at(e), ca * d);
    }
    st_row<VEC>(out, rp, xo);
  }
}

// The y and z terms of one row: out += m * sum_{a = y, z} (D1_a psi_a +
// zeta_a), zeta_a updated, VEC consecutive x nodes per lane (nx % VEC == 0).
// Per node the operations of cpml_fix_kernel without its x part.
template <int VEC>
__device__ __forceinline__ void fix_row(const CpmlArgs &c, const float *cur, const float *m, float *out, int y, int z,
                                        uint32_t xo) {
  const unsigned nx = c.nx, ny = c.ny, W2 = 2u * c.W;
  const size_t o = (static_cast<size_t>(z) * ny + static_cast<unsigned>(y)) * nx;
  const float *row = cur + o;
  const rsrc_t ro = row_at(out + o, true, nx);
  const Row<VEC> mv = ld_row<VEC>(row_at(m + o, true, nx), xo);
  const Row<VEC> ov = ld_row<VEC>(ro, xo);
  const Row<VEC> cc = ld_row<VEC>(row_at(row, true, nx), xo);
  float extra[kRowNodes];
#pragma unroll
  for (int e = 0; e < kRowNodes; ++e) extra[e] = 0.f;
#pragma unroll
  for (int a = 1; a < 3; ++a) {
    const int i = a == 1 ? y : z, n = a == 1 ? c.ny : c.nz;
    if (i >= c.W + R && i < n - c.W - R) continue;  // psi_a and zeta_a vanish this far in
    const size_t stride = a == 1 ? nx : static_cast<size_t>(nx) * ny;
    // slab row of slab index s: y: (z, s), z: (s, y)
    auto slab = [&](int sidx) {
      return (a == 1 ? static_cast<size_t>(z) * W2 + sidx : static_cast<size_t>(sidx) * ny + static_cast<unsigned>(y)) * nx;
    };
    const int s = slab_index(i, n, c.W);
    Row<VEC> pp[R], pm[R], up[R], dn[R];
#pragma unroll
    for (int k = 1; k <= R; ++k) {
      const int sp = slab_index(i + k, n, c.W), sm = slab_index(i - k, n, c.W);
      pp[k - 1] = ld_row<VEC>(row_at(c.psi[a] + slab(sp < 0 ? 0 : sp), sp >= 0, nx), xo);
      pm[k - 1] = ld_row<VEC>(row_at(c.psi[a] + slab(sm < 0 ? 0 : sm), sm >= 0, nx), xo);
    }
    if (s < 0) {  // beyond the layer: D1 psi alone
#pragma unroll
      for (int e = 0; e < kRowNodes; ++e) {
        float dpsi = 0.f;
#pragma unroll
        for (int k = 1; k <= R; ++k)
          dpsi = fmaf(c.d1w[a][k - 1], pp[k - 1].at(e) - pm[k - 1].at(e), dpsi);
        extra[e] += dpsi;
      }
      continue;
    }
#pragma unroll
    for (int k = 1; k <= R; ++k) {
      up[k - 1] = ld_row<VEC>(row_at(row + k * stride, i + k < n, nx), xo);
      dn[k - 1] = ld_row<VEC>(row_at(row - k * stride, i - k >= 0, nx), xo);
    }
    const rsrc_t rz = row_at(c.zeta[a] + slab(s), true, nx);
    const Row<VEC> zv = ld_row<VEC>(rz, xo);
    const float ca = c.ca[a][i], cb = c.cb[a][i];
    float zn[kRowNodes];
#pragma unroll
    for (int e = 0; e < kRowNodes; ++e) {
      const float u = cc.at(e);
      float dpsi = 0.f, d2 = 0.f;  // d2: second differences from the centre (no large centre term)
#pragma unroll
      for (int k = 1; k <= R; ++k) {
        dpsi = fmaf(c.d1w[a][k - 1], pp[k - 1].at(e) - pm[k - 1].at(e), dpsi);
        d2 = fmaf(c.d2w[a][k], (up[k - 1].at(e) - u) + (dn[k - 1].at(e) - u), d2);
      }
      zn[e] = fmaf(cb, zv.at(e), ca * (d2 + dpsi));
      extra[e] += dpsi + zn[e];
    }
    st_row<VEC>(zn, rz, xo);
  }
  float res[kRowNodes];
#pragma unroll
  for (int e = 0; e < kRowNodes; ++e) res[e] = fmaf(mv.at(e), extra[e], ov.at(e));
  st_row<VEC>(res, ro, xo);
}

// A lane's vectors of a row as offsets into a resource of several rows: past
// the row's end, out of every resource.
template <int VEC> struct RowOff {
  uint32_t o[kRowNodes / VEC];
  __device__ RowOff(uint32_t xo, unsigned nx) {
#pragma unroll
    for (int k = 0; k < kRowNodes / VEC; ++k) {
      const uint32_t x = xo + k * (256u * VEC);
      o[k] = x < nx * 4u ? x : kOOB;
    }
  }
  // the row at byte `at` (zeros if not in)
  __device__ Row<VEC> ld(rsrc_t r, uint32_t at, bool in) const {
    Row<VEC> out;
#pragma unroll
    for (int k = 0; k < kRowNodes / VEC; ++k) out.v[k] = ld_words<VEC * 4, 0>(r, in ? o[k] : kOOB, in ? at : 0u);
    return out;
  }
  __device__ void st(const float *v, rsrc_t r, uint32_t at) const {
#pragma unroll
    for (int k = 0; k < kRowNodes / VEC; ++k) st_words<VEC * 4, 0>(row_put<kF32, VEC>(v + k * VEC), r, o[k], at);
  }
};

// The same for G consecutive rows along axis A (1: y, 2: z) that have that
// axis' terms alone, each psi and A^n row of their window loaded once.  One
// resource per array (the window's rows or the axis' slab, each below 2^31
// bytes) and a scalar offset per row: a resource per row spilled 300 scalar
// registers.
template <int VEC, int A, int G>
__device__ __forceinline__ void fix_rows(const CpmlArgs &c, const float *cur, const float *m, float *out, int y, int z,
                                         uint32_t xo) {
  const unsigned nx = c.nx, ny = c.ny, W2 = 2u * c.W;
  const int i0 = A == 1 ? y : z, n = A == 1 ? c.ny : c.nz;
  const size_t o = (static_cast<size_t>(z) * ny + static_cast<unsigned>(y)) * nx;
  const uint32_t row = nx * 4u, stride = A == 1 ? row : row * ny;
  const RowOff<VEC> off(xo, nx);
  // byte of the row of slab index s: y: (z, s), z: (s, y)
  auto slab = [&](int s) { return (A == 1 ? static_cast<uint32_t>(z) * W2 + s : s * ny + static_cast<uint32_t>(y)) * row; };
  const uint32_t slab_bytes = (A == 1 ? static_cast<uint32_t>(c.nz) : ny) * W2 * row;
  const rsrc_t rs = make_rsrc(c.psi[A], slab_bytes), rz = make_rsrc(c.zeta[A], slab_bytes);
  const int b = max(i0 - R, 0), top = min(i0 + G - 1 + R, n - 1);  // the window's rows within the grid
  const rsrc_t ru = make_rsrc(cur + o - static_cast<size_t>(i0 - b) * (stride / 4u), static_cast<uint32_t>(top - b) * stride + row);
  const rsrc_t rm = make_rsrc(m + o, (G - 1) * stride + row), ro = make_rsrc(out + o, (G - 1) * stride + row);
  bool layer = false;  // rows with zeta_a (and a second difference) among them
#pragma unroll
  for (int j = 0; j < G; ++j) layer |= slab_index(i0 + j, n, c.W) >= 0;
  Row<VEC> ps[G + 2 * R], u[G + 2 * R], mv[G], ov[G], zv[G];
#pragma unroll
  for (int k = 0; k < G + 2 * R; ++k) {
    const int i = i0 + k - R, s = slab_index(i, n, c.W);
    ps[k] = off.ld(rs, slab(s), s >= 0);
    u[k] = off.ld(ru, static_cast<uint32_t>(i - b) * stride, layer && i >= 0 && i < n);
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int s = slab_index(i0 + j, n, c.W);
    zv[j] = off.ld(rz, slab(s), s >= 0);
    mv[j] = off.ld(rm, j * stride, true);
    ov[j] = off.ld(ro, j * stride, true);
  }
#pragma unroll
  for (int j = 0; j < G; ++j) {
    const int s = slab_index(i0 + j, n, c.W);
    const float ca = c.ca[A][i0 + j], cb = c.cb[A][i0 + j];
    float zn[kRowNodes], res[kRowNodes];
#pragma unroll
    for (int e = 0; e < kRowNodes; ++e) {
      const float cc = u[j + R].at(e);
      float dpsi = 0.f, d2 = 0.f;  // d2: second differences from the centre (no large centre term)
#pragma unroll
      for (int k = 1; k <= R; ++k) {
        dpsi = fmaf(c.d1w[A][k - 1], ps[j + R + k].at(e) - ps[j + R - k].at(e), dpsi);
        d2 = fmaf(c.d2w[A][k], (u[j + R + k].at(e) - cc) + (u[j + R - k].at(e) - cc), d2);
      }
      zn[e] = fmaf(cb, zv[j].at(e), ca * (d2 + dpsi));
      const float extra = 0.f + (s < 0 ? dpsi : dpsi + zn[e]);  // beyond the layer: D1 psi alone
      res[e] = fmaf(mv[j].at(e), extra, ov[j].at(e));
    }
    if (s >= 0) off.st(zn, rz, slab(s));
    off.st(res, ro, j * stride);
  }
}

// The y and z terms after the step with the x part fused in, over the rows of
// the first two parts of the (W + R)-node shell (the other nodes get no y or z
// term).  A wavefront takes kFixRows rows along the axis of its layer: with
// one row each it was bound by its loads through L1 and L2, 16 neighbour rows
// of psi and A^n for every row, of which neighbouring rows share most: four
// rows together need 24 where they loaded 68.  Rows with both terms (edges of the box) and groups across the end of a
// layer go row by row.  Measured, a whole CPML step, one row and four rows per
// wavefront: 512^3 647 -> 626 us, 401x333x301 362 -> 355 us, 256^3 and
// 300x99x174 equal.
constexpr unsigned kFixRows = 4;
template <int VEC>
__global__ void __launch_bounds__(256) cpml_fix_yz_kernel(CpmlArgs c, ShellWork P, const float *__restrict__ cur,
                                                          const float *__restrict__ m, float *out) {
  const ShellAt at = shell_at(P);
  if (at.part >= 2) return;
  const Shell &S = P.S;
  const uint32_t xo = at.seg * (64u * kRowNodes * 4u) + (threadIdx.x & 63u) * (VEC * 4u);
  const int y = at.y, z = at.z;
  const unsigned k1 = at.k + kFixRows - 1, count = at.part == 0 ? S.cz : S.cy;
  const int E = c.W + R;
  if (at.part == 0) {
    if (k1 < count && S.z_at(k1) == z + kFixRows - 1 && y >= E && y < c.ny - E)
      return fix_rows<VEC, 2, kFixRows>(c, cur, m, out, y, z, xo);
  } else if (k1 < count && S.y_at(k1) == y + kFixRows - 1) {
    return fix_rows<VEC, 1, kFixRows>(c, cur, m, out, y, z, xo);
  }
  for (unsigned k = at.k; k <= k1 && k < count; ++k)
    fix_row<VEC>(c, cur, m, out, at.part == 0 ? y : static_cast<int>(S.y_at(k)),
                 at.part == 0 ? static_cast<int>(S.z_at(k)) : z, xo);
}

// After the plain step: one thread per node within W + R of a face adds the
// terms of all three axes.
__global__ void __launch_bounds__(256) cpml_fix_kernel(CpmlArgs c, const float *__restrict__ cur,
                                                       const float *__restrict__ m, float *out) {
  const Shell S(c.W + R, c.nx, c.ny, c.nz);
  const unsigned t = blockIdx.x * 256u + threadIdx.x;
  if (t >= S.count()) return;
  int x, y, z;
  S.node(t, x, y, z);
  const unsigned o = (static_cast<unsigned>(z) * c.ny + y) * c.nx + x;
  float extra = 0.f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const AxisAt A = axis_at(c, a, x, y, z);
    if (A.i >= c.W + R && A.i < A.n - c.W - R) continue;  // psi_a and zeta_a vanish this far in
    float dpsi = 0.f;
#pragma unroll
    for (int k = 1; k <= R; ++k) dpsi = fmaf(c.d1w[a][k - 1], psi_k(c, a, A, k) - psi_k(c, a, A, -k), dpsi);
    const int s = slab_index(A.i, A.n, c.W);
    if (s < 0) {
      extra += dpsi;
      continue;
    }
    const float cc = cur[o];
    float d2 = 0.f;
#pragma unroll
    for (int k = 1; k <= R; ++k) d2 = fmaf(c.d2w[a][k], (cur_k(cur, o, A, k) - cc) + (cur_k(cur, o, A, -k) - cc), d2);
    float *ze = c.zeta[a] + A.slab_rest + static_cast<unsigned>(s) * A.slab_stride;
    const float zn = fmaf(c.cb[a][A.i], *ze, c.ca[a][A.i] * (d2 + dpsi));
    *ze = zn;
    extra += dpsi + zn;
  }
  out[o] = fmaf(m[o], extra, out[o]);
}

// ------------------------------------------------------------ utilities

// ------------------------------------------------------------ conversion passes
//
// Copies, conversions and reductions between the caller's arrays (rows of nx
// nodes) and the workspace's fields (rows of their pitch): a lane takes four
// consecutive nodes, as one vector on both sides.  A pass that sets a field
// goes through the field's vectors and loads the caller's nodes where they
// start, at any element (which a global access may); the columns that pad a row
// become zero.  A pass that reads one goes through the caller's vectors; one
// that lies across the end of a row takes the two parts from two loads.  Arrays
// without row padding count as one row.  Bound by memory: one access per lane
// and array in many short workgroups, the form that streams fastest here.
// Against one node per lane and access in a strided loop, 1024^3 bf16: reading a
// field 1940 -> 1030 us, its maximum 1200 -> 800 us, encoding it 1500 -> 1105 us.
// The set-up of m at 256^3, which queued two atomics per workgroup on one line:
// 378 -> 40 us.  Rows of a vector each, a wavefront per row and single accesses
// in padded rows, took 2 to 14 times as long where rows are short or padded: A^{n-1}
// of 4x2048x2048 f16 783 -> 40 us, reading 33x896x896 f32 87 -> 41 us, writing it
// 133 -> 44 us, and a snapshot of 301x512x512 f16, then copied by
// hipMemcpy2DAsync, 1208 -> 227 us.

// n / d for n d < 2^64.
struct FastDiv64 {
  unsigned d;
  uint64_t m;
  explicit FastDiv64(unsigned div = 1) : d(div), m(~uint64_t(0) / div + 1) {}  // d = 1: m = 0, not used
  __host__ __device__ uint64_t operator()(uint64_t n) const {
    return d == 1 ? n : static_cast<uint64_t>((static_cast<unsigned __int128>(n) * m) >> 64);
  }
};

struct RowMap {
  size_t total;     // nodes of the caller's array
  size_t nvec;      // vectors gone through: of the field (set), of the caller's array (read)
  unsigned nx, pitch;
  FastDiv64 row;    // vectors per row of the field (set), nodes per row of the caller's array (read)
  FastDiv in_row;   // the same for indices within a row and a wavefront
};

// Four values of type T at an address aligned to ALIGN bytes, or the first n
// of them (single accesses).
template <int ALIGN, bool NT, typename T> __device__ __forceinline__ void get4(const T *p, T (&v)[4]) {
  typedef T four __attribute__((ext_vector_type(4), aligned(ALIGN)));
  const four *q = reinterpret_cast<const four *>(p);
  const four t = NT ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = t[e];
}
template <int ALIGN, bool NT, typename T> __device__ __forceinline__ void put4(T *p, const T (&v)[4]) {
  typedef T four __attribute__((ext_vector_type(4), aligned(ALIGN)));
  four t;
#pragma unroll
  for (int e = 0; e < 4; ++e) t[e] = v[e];
  four *q = reinterpret_cast<four *>(p);
  if constexpr (NT) __builtin_nontemporal_store(t, q);
  else *q = t;
}
template <int ALIGN, bool NT, typename T> __device__ __forceinline__ void get4(const T *p, T (&v)[4], unsigned n) {
  typedef T one __attribute__((aligned(ALIGN)));
  if (n >= 4u) return get4<ALIGN, NT>(p, v);
#pragma unroll
  for (unsigned e = 0; e < 4u; ++e) v[e] = e < n ? reinterpret_cast<const one *>(p)[e] : T(0);
}
template <int ALIGN, bool NT, typename T> __device__ __forceinline__ void put4(T *p, const T (&v)[4], unsigned n) {
  typedef T one __attribute__((aligned(ALIGN)));
  if (n >= 4u) return put4<ALIGN, NT>(p, v);
#pragma unroll
  for (unsigned e = 0; e < 4u; ++e)
    if (e < n) reinterpret_cast<one *>(p)[e] = v[e];
}
// Four values encoded in storage type S.
template <int S> __device__ __forceinline__ void encode4(const float (&v)[4], typename Codec<S>::raw (&r)[4]) {
  if constexpr (S == kF32) {
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = v[e];
  } else {
    const Words<8> w = row_put<S, 4>(v);
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = static_cast<uint16_t>(w.w[e >> 1] >> (16 * (e & 1)));
  }
}

// Passes that set a field or reduce over the caller's array.  Op::in(u, v, n):
// n of four nodes from index u of the caller's array; Op::set(f, v, n, k): k of
// four nodes of the field from index f, which hold v[0 .. n) and zeros;
// Op::finish() once per thread.
template <bool FLAT, class Op>
__global__ void __launch_bounds__(256) set_kernel(Op op, RowMap map) {
  const unsigned lane = threadIdx.x & 63u;
  const unsigned wave = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6));
  for (size_t t0 = (static_cast<size_t>(blockIdx.x) * 4u + wave) * 64u; t0 < map.nvec; t0 += static_cast<size_t>(gridDim.x) * 256u) {
    if (t0 + lane >= map.nvec) break;
    const size_t f = (t0 + lane) * 4u;
    size_t u = f;
    unsigned n = 4u;
    if constexpr (!FLAT) {
      const uint64_t r0 = map.row(t0);
      const unsigned i = static_cast<unsigned>(t0 - r0 * map.row.d) + lane, k = map.in_row(i);
      const unsigned col = (i - k * map.in_row.d) * 4u;
      u = (r0 + k) * map.nx + col;
      n = min(4u, map.nx - col);
    }
    typename Op::T v[4];
    if (FLAT && (t0 + 64u) * 4u <= map.total) {  // the whole wavefront: no checks per lane
      op.in(u, v, 4u);
      op.set(f, v, 4u, 4u);
      continue;
    }
    // the nodes past a row's end are the next row's, but for the array's last
    const unsigned have = static_cast<unsigned>(min(map.total - u, size_t(4)));
    op.in(u, v, have);
    if constexpr (FLAT) op.set(f, v, have, have);
    else op.set(f, v, n, 4u);
  }
  op.finish();
}

// Passes that read a field.  Op::at(f, v): four stored nodes of the field from
// index f; Op::out(u, v, r0, k, col, n): n of them to index u of the caller's
// array, the first one node col of row r0 + k, r0 the same for the wavefront
// (FLAT: row 0, col = u).
template <bool FLAT, class Op>
__global__ void __launch_bounds__(256) read_kernel(Op op, RowMap map) {
  const unsigned lane = threadIdx.x & 63u;
  const unsigned wave = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6));
  for (size_t t0 = (static_cast<size_t>(blockIdx.x) * 4u + wave) * 64u; t0 < map.nvec; t0 += static_cast<size_t>(gridDim.x) * 256u) {
    if (t0 + lane >= map.nvec) break;
    const size_t u = (t0 + lane) * 4u;
    typename Op::Raw v;
    uint64_t r0 = 0;
    unsigned k = 0;
    size_t col = u;
    if constexpr (FLAT) {
      op.at(u, v);
    } else {
      const size_t u0 = t0 * 4u;
      r0 = map.row(u0);
      const unsigned i = static_cast<unsigned>(u0 - r0 * map.row.d) + 4u * lane;
      k = map.in_row(i);
      col = i - k * map.in_row.d;
      op.at((r0 + k) * map.pitch + col, v);
      const unsigned n = static_cast<unsigned>(map.nx - col);
      if (n < 4u) {
        typename Op::Raw w;
        op.at((r0 + k + 1) * map.pitch - n, w);
        v.from(w, n);
      }
    }
    op.out(u, v, r0, k, col, static_cast<unsigned>(min(map.total - u, size_t(4))));
  }
}

// Four stored values of each of K fields.
template <typename T, int K> struct Raw4 {
  T v[K][4];
  __device__ void from(const Raw4 &o, unsigned n) {  // the values from the nth on are o's
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (unsigned e = 1; e < 4u; ++e) v[k][e] = e < n ? v[k][e] : o.v[k][e];
  }
};

// lo, hi: smallest and largest of a value per thread over the workgroup;
// thread 0 gets them.
__device__ __forceinline__ void block_range(float &lo, float &hi, int &bad) {
  __shared__ float smin[4], smax[4];
  __shared__ int sbad[4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = fminf(lo, __shfl_xor(lo, off, 64));
    hi = fmaxf(hi, __shfl_xor(hi, off, 64));
    bad |= __shfl_xor(bad, off, 64);
  }
  const int w = static_cast<int>(threadIdx.x) >> 6;
  if ((threadIdx.x & 63) == 0) {
    smin[w] = lo;
    smax[w] = hi;
    sbad[w] = bad;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    lo = fminf(lo, smin[k]);
    hi = fmaxf(hi, smax[k]);
    bad |= sbad[k];
  }
}
// Raise (lower) a shared word, whose atomics queue at 11 ns each, only where
// the value read says that it would change.
__device__ __forceinline__ void raise(uint32_t *p, uint32_t v) {
  if (v > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, v);
}
__device__ __forceinline__ void lower(uint32_t *p, uint32_t v) {
  if (v < __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(p, v);
}

// m = (v dt)^2 (not written where m is null), the velocity's range and whether
// every value is finite and positive.
struct InitM {
  using T = float;
  const float *vel;
  float *m;
  float dt;
  StepState *st;
  float lo = __builtin_huge_valf(), hi = 0.f;
  int bad = 0;
  __device__ void in(size_t u, float (&v)[4], unsigned n) { get4<4, false>(vel + u, v, n); }
  __device__ void set(size_t f, const float (&v)[4], unsigned n, unsigned k) {
    float o[4];
#pragma unroll
    for (unsigned e = 0; e < 4u; ++e) {
      const float t = v[e] * dt;
      o[e] = e < n ? t * t : 0.f;
      if (e < n) {
        if (!(v[e] > 0.f) || !(v[e] < __builtin_huge_valf())) bad = 1;
        lo = fminf(lo, v[e]);
        hi = fmaxf(hi, v[e]);
      }
    }
    if (m) put4<16, false>(m + f, o, k);
  }
  __device__ void finish() {
    block_range(lo, hi, bad);
    if (threadIdx.x == 0) {
      if (bad) atomicOr(&st->flags, 2u);
      if (lo > 0.f) lower(&st->vmin_bits, __float_as_uint(lo));
      raise(&st->vmax_bits, __float_as_uint(fmaxf(hi, 0.f)));
    }
  }
};

struct EncodeM16 {
  using T = float;
  const float *vel;
  uint16_t *codes;
  float dt, m_lo, m_step;
  __device__ void in(size_t u, float (&v)[4], unsigned n) { get4<4, false>(vel + u, v, n); }
  __device__ void set(size_t f, const float (&v)[4], unsigned n, unsigned k) {
    uint16_t c[4];
#pragma unroll
    for (unsigned e = 0; e < 4u; ++e) {
      const float t = v[e] * dt;
      const float q = m_step > 0.f ? rintf((t * t - m_lo) / m_step) : 0.f;
      c[e] = e < n ? static_cast<uint16_t>(fminf(fmaxf(q, 0.f), 65535.f)) : uint16_t(0);
    }
    put4<8, false>(codes + f, c, k);
  }
  __device__ void finish() {}
};

// Setting a 16-bit stored field from float32 values (wave_write_field): the
// field's maximum record of step n first holds max |x| (float bits; the
// values are non-negative, so unsigned order is float order), the encode
// uses the exponent the step kernel's rule gives for that bound, and the
// record then takes the largest stored magnitude, with the exponent beside it.
__global__ void scale_record_clear_kernel(StepState *st, uint32_t *slots, int v_field) {
  if (threadIdx.x == 0) (v_field ? st->amax_v : st->amax)[st->n & 3] = 0u;
  if (threadIdx.x < kMaxSlots) slots[max_slot(st->n, threadIdx.x) + v_field] = 0u;
}

struct AbsMax {
  using T = float;
  const float *x;
  StepState *st;
  int v_field;
  float mx = 0.f;
  __device__ void in(size_t u, float (&v)[4], unsigned n) { get4<4, false>(x + u, v, n); }
  __device__ void set(size_t, const float (&v)[4], unsigned n, unsigned) {
#pragma unroll
    for (unsigned e = 0; e < 4u; ++e)
      if (e < n) mx = fmaxf(mx, fabsf(v[e]));
  }
  __device__ void finish() {
    float lo = 0.f;
    int bad = 0;
    block_range(lo, mx, bad);
    if (threadIdx.x == 0) raise(&(v_field ? st->amax_v : st->amax)[st->n & 3], __float_as_uint(mx));
  }
};

template <int S> struct EncodeField {
  using T = float;
  const float *x;
  typename Codec<S>::raw *dst;
  const StepState *st;
  int v_field;
  __device__ void in(size_t u, float (&v)[4], unsigned n) { get4<4, true>(x + u, v, n); }
  __device__ void set(size_t f, const float (&v)[4], unsigned n, unsigned k) {
    const float sc = exp2i(scale_exponent(__uint_as_float((v_field ? st->amax_v : st->amax)[st->n & 3])));
    float s[4];
    typename Codec<S>::raw r[4];
#pragma unroll
    for (unsigned e = 0; e < 4u; ++e) s[e] = e < n ? v[e] * sc : 0.f;
    encode4<S>(s, r);
    put4<8, false>(dst + f, r, k);
  }
  __device__ void finish() {}
};

template <int S>
__global__ void scale_record_kernel(StepState *st, int v_field) {
  if (threadIdx.x != 0) return;
  const int slot = st->n & 3;
  uint32_t *rec = v_field ? st->amax_v : st->amax;
  const float bound = __uint_as_float(rec[slot]);
  const int e = scale_exponent(bound);
  rec[slot] = __float_as_uint(fabsf(Codec<S>::dec(Codec<S>::enc(bound * exp2i(e)))));
  (v_field ? st->exps_v : st->exps)[slot] = e;
}

// Values as they are into a field, from an array that starts at any multiple
// of ALIGN bytes (float32 between two fields too, of which a checkpoint starts at
// any element).  NT: past the cache, for arrays that with the field overflow
// the 256 MB last-level cache (256x512x512 100 -> 87 us; 16x1024x1024, within it, 34 -> 31 us
// without).
template <typename V, int ALIGN, bool NT = false> struct CopyIn {
  using T = V;
  const V *x;
  V *dst;
  __device__ void in(size_t u, V (&v)[4], unsigned n) { get4<ALIGN, NT>(x + u, v, n); }
  __device__ void set(size_t f, const V (&v)[4], unsigned n, unsigned k) {
    V o[4];
#pragma unroll
    for (unsigned e = 0; e < 4u; ++e) o[e] = e < n ? v[e] : V(0);
    put4<sizeof(V), false>(dst + f, o, k);
  }
  __device__ void finish() {}
};

// The reverse.
template <typename V, int ALIGN> struct CopyOut {
  using Raw = Raw4<V, 1>;
  const V *src;
  V *dst;
  __device__ void at(size_t f, Raw &r) { get4<sizeof(V), false>(src + f, r.v[0]); }
  __device__ void out(size_t u, const Raw &r, uint64_t, unsigned, size_t, unsigned n) { put4<ALIGN, true>(dst + u, r.v[0], n); }
};

template <int S> struct Decode {
  using raw = typename Codec<S>::raw;
  using Raw = Raw4<raw, 1>;
  const raw *src;
  float *dst;
  const StepState *st;
  int slot_off, v_field;
  __device__ void at(size_t f, Raw &r) { get4<sizeof(raw), false>(src + f, r.v[0]); }
  __device__ void out(size_t u, const Raw &r, uint64_t, unsigned, size_t, unsigned n) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = Codec<S>::dec(r.v[0][e]);
    if constexpr (S != kF32) {
      const int slot = (st->n + slot_off) & 3;
      const float inv = exp2i(-(v_field ? st->exps_v[slot] : st->exps[slot]));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= inv;
    }
    put4<4, true>(dst + u, v, n);
  }
};

// A^{n-1} = (A^n - V^n) / g from the 16-bit velocity-form pair.
template <int S> struct DecodePrev {
  using raw = typename Codec<S>::raw;
  using Raw = Raw4<raw, 2>;
  const raw *fa, *fv;
  float *dst;
  const float *gx, *gy, *gz;
  FastDiv64 nx, ny;
  FastDiv ny32;
  const StepState *st;
  __device__ void at(size_t f, Raw &r) {
    get4<sizeof(raw), false>(fa + f, r.v[0]);
    get4<sizeof(raw), false>(fv + f, r.v[1]);
  }
  __device__ float gyz(uint64_t r0, unsigned k) const {  // the step kernel's association; gz goes on past the grid
    const uint64_t z = ny(r0);
    const unsigned y = static_cast<unsigned>(r0 - z * ny.d) + k, over = ny32(y);
    return gy[y - over * ny32.d] * gz[z + over];
  }
  __device__ void out(size_t u, const Raw &r, uint64_t r0, unsigned k, size_t col, unsigned n) {
    const int slot = st->n & 3;
    const float ia = exp2i(-st->exps[slot]), iv = exp2i(-st->exps_v[slot]);
    if (col >= nx.d) {  // counted through the rows
      r0 = nx(col);
      col -= r0 * nx.d;
    }
    float v[4], g[4], gr = gyz(r0, k);
    if (col + 4u <= nx.d) {
      get4<4, false>(gx + col, g);
#pragma unroll
      for (int e = 0; e < 4; ++e) g[e] *= gr;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (col == nx.d) {
          col = 0;
          gr = gyz(r0, ++k);
        }
        g[e] = gx[col++] * gr;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (Codec<S>::dec(r.v[0][e]) * ia - Codec<S>::dec(r.v[1][e]) * iv) / g[e];
    put4<4, true>(dst + u, v, n);
  }
};

// dJ/dv = 2 img dt / sqrt(m)
struct GradFinal {
  using Raw = Raw4<float, 2>;
  const float *img, *m;
  float dt;
  float *grad;
  __device__ void at(size_t f, Raw &r) {
    get4<4, false>(img + f, r.v[0]);
    get4<4, false>(m + f, r.v[1]);
  }
  __device__ void out(size_t u, const Raw &r, uint64_t, unsigned, size_t, unsigned n) {
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = 2.f * r.v[0][e] * dt / sqrtf(r.v[1][e]);
    put4<4, true>(grad + u, v, n);
  }
};

// One access per lane, within the 2^32 threads of a launch; a reduction ends in
// an atomic per workgroup: 8 workgroups per CU read the array.
dim3 vec_grid(size_t nvec, size_t most) {
  const size_t want = (nvec + 255) / 256;
  return dim3(static_cast<unsigned>(want < most ? want : most));
}
constexpr size_t kMostGroups = 1u << 22;

template <class Op> hipError_t launch_set(Op op, const GridRows &g, bool reduces, hipStream_t s) {
  RowMap map;
  map.total = g.rows * g.nx;
  map.nvec = (g.rows * g.pitch + 3) / 4;  // padded pitches are whole vectors
  map.nx = g.nx;
  map.pitch = g.pitch;
  map.row = FastDiv64(map.pitch > 4u ? map.pitch / 4u : 1u);
  map.in_row = FastDiv(map.row.d);
  const dim3 grid = vec_grid(map.nvec, reduces ? 2048 : kMostGroups), b(256);
  if (g.pitch == g.nx) hipLaunchKernelGGL((set_kernel<true, Op>), grid, b, 0, s, op, map);
  else hipLaunchKernelGGL((set_kernel<false, Op>), grid, b, 0, s, op, map);
  return hipGetLastError();
}

// by_row: the operation needs rows and columns, which rows of whole vectors give
// it without a division per lane.  The field's allocation goes on for a vector
// past its last node (padding planes).
template <class Op> hipError_t launch_read(Op op, const GridRows &g, bool by_row, hipStream_t s) {
  RowMap map;
  map.total = g.rows * g.nx;
  map.nvec = (map.total + 3) / 4;
  map.nx = g.nx;
  map.pitch = g.pitch;
  map.row = FastDiv64(map.nx);
  map.in_row = FastDiv(map.nx);
  const dim3 grid = vec_grid(map.nvec, kMostGroups), b(256);
  if (g.pitch == g.nx && !(by_row && g.nx % 4 == 0)) hipLaunchKernelGGL((read_kernel<true, Op>), grid, b, 0, s, op, map);
  else hipLaunchKernelGGL((read_kernel<false, Op>), grid, b, 0, s, op, map);
  return hipGetLastError();
}

__global__ void bump_kernel(StepState *st, int count, const uint32_t *slots) {  // one wavefront
  const int n = st->n + count;
  if (slots) {
    uint32_t ma = st->amax[n & 3], mv = st->amax_v[n & 3];
    max_slots(slots, n, ma, mv);
    if (threadIdx.x == 0) {
      st->amax[n & 3] = ma;
      st->amax_v[n & 3] = mv;
    }
  }
  if (threadIdx.x == 0) st->n = n;
}

__global__ void set_n_kernel(StepState *st, int n) {
  if (threadIdx.x == 0) st->n = n;
}

__global__ void reset_state_kernel(StepState *st, uint32_t *slots) {
  const int t = threadIdx.x;
  if (slots)
    for (int k = t; k < 4 * kMaxSlots * 2; k += 64) slots[max_slot(k >> 5, (k >> 1) & 15) + (k & 1)] = 0u;
  if (t == 0) {
    st->n = 0;
    st->flags = 0u;
  }
  if (t < 4) {
    st->amax[t] = 0u;
    st->exps[t] = 0;
    st->amax_v[t] = 0u;
    st->exps_v[t] = 0;
  }
}

template <int S>
__global__ void gather_kernel(const typename Codec<S>::raw *__restrict__ f, const int64_t *__restrict__ lin,
                              int nrec, float *__restrict__ traces, const StepState *st, int k) {
  const int n = st->n + k;
  const int e = S == kF32 ? 0 : st->exps[(n + 1) & 3];
  const float inv = exp2i(-e);
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < nrec) traces[static_cast<size_t>(n) * nrec + r] = Codec<S>::dec(f[lin[r]]) * inv;
}

// Adjoint injection at an irregular receiver list: one thread per distinct
// receiver node adds g m times the sum of that node's residuals, taken in
// receiver order.  Each node is written by one thread and duplicates are
// summed in a fixed order, so the result does not depend on scheduling.
__global__ void scatter_kernel(float *f, const int64_t *__restrict__ node, const int32_t *__restrict__ off,
                               const int32_t *__restrict__ ord, int nnode, int nrec, const float *__restrict__ m,
                               const float *__restrict__ gnode, const float *__restrict__ resid, int row) {
  const int u = blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= nnode) return;
  const float *rr = resid + static_cast<size_t>(row) * nrec;
  float sum = 0.f;
  for (int j = off[u]; j < off[u + 1]; ++j) sum += rr[ord[j]];
  const int64_t p = node[u];
  f[p] = fmaf(gnode[u] * m[p], sum, f[p]);
}

template <int S>
__global__ void finite_kernel(const typename Codec<S>::raw *__restrict__ f, size_t n, StepState *st) {
  int bad = 0;
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const float v = Codec<S>::dec(f[i]);
    if (!(fabsf(v) < __builtin_huge_valf())) bad = 1;
  }
  if (bad) atomicOr(&st->flags, 1u);
}

// Field values to time candidate configurations on (hash of the node index):
// float32 in [-1, 1), 16-bit codes of magnitude below 2^10.
template <int S>
__global__ void noise_kernel(typename Codec<S>::raw *__restrict__ f, size_t n, uint32_t seed) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x) {
    uint32_t h = static_cast<uint32_t>(i) * 2654435761u + seed;
    h = (h ^ (h >> 15)) * 2246822519u;
    h ^= h >> 13;
    const float v = static_cast<float>(static_cast<int32_t>(h)) * 0x1p-31f;
    f[i] = Codec<S>::enc(S == kF32 ? v : v * 1024.f);
  }
}

__global__ void zero_kernel(uint4 *p, size_t n16, uint8_t *tail, size_t ntail) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n16;
       i += static_cast<size_t>(gridDim.x) * blockDim.x)
    p[i] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

unsigned grid_for(size_t n, unsigned block) {
  const size_t want = (n + block - 1) / block;
  const size_t cap = 256 * 64;  // enough workgroups to cover all CUs many times over
  return static_cast<unsigned>(want < 1 ? 1 : (want > cap ? cap : want));
}
}  // namespace

int variant_count() { return kNumVariants; }

int step_blocks_per_cu(int storage, int variant, bool cpml) {
  if (variant < 0 || variant >= kNumVariants) return 1;
  switch (storage) {
    case kF32: return blocks_variant_f32(variant, cpml);
    case kF16: return blocks_variant_f16(variant);
    case kBF16: return blocks_variant_bf16(variant);
    default: return 1;
  }
}

Variant variant_info(int v) { return kVariants[v]; }

bool variant_fuses_cpml(int v) {
  switch (v) {
#define WAVE_VARIANT_CASE(id, fam, by, ry, pd, vec, lx) \
  case id: return fam == 0 && fuses_cpml<ry, vec>();
    WAVE_VARIANTS(WAVE_VARIANT_CASE)
#undef WAVE_VARIANT_CASE
    default: return false;
  }
}

hipError_t launch_step(int storage, int variant, bool adjoint, const StepArgs &a, hipStream_t s) {
  if (variant < 0 || variant >= kNumVariants) return hipErrorInvalidValue;
  if (adjoint) {
    if (storage != kF32) return hipErrorInvalidValue;
    return launch_variant_adj(variant, a, s);
  }
  switch (storage) {
    case kF32: return a.lap ? launch_variant_lap(variant, a, s) : launch_variant_f32(variant, a, s);
    case kF16: return a.m16 ? launch_variant_f16m(variant, a, s) : launch_variant_f16(variant, a, s);
    case kBF16: return a.m16 ? launch_variant_bf16m(variant, a, s) : launch_variant_bf16(variant, a, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_init_m(const float *vel, float *m, const GridRows &g, float dt, StepState *st, hipStream_t s) {
  return launch_set(InitM{vel, m, dt, st}, g, true, s);
}

hipError_t launch_encode_m16(const float *vel, uint16_t *codes, const GridRows &g, float dt, float m_lo, float m_step,
                             hipStream_t s) {
  return launch_set(EncodeM16{vel, codes, dt, m_lo, m_step}, g, false, s);
}

hipError_t launch_encode_field(int storage, const float *x, void *dst, const GridRows &g, StepState *st,
                              uint32_t *slots, bool v_field, hipStream_t s) {
  if (storage != kF16 && storage != kBF16) return hipErrorInvalidValue;
  const int vf = v_field ? 1 : 0;
  hipLaunchKernelGGL(scale_record_clear_kernel, dim3(1), dim3(64), 0, s, st, slots, vf);
  hipError_t e = launch_set(AbsMax{x, st, vf}, g, true, s);
  if (e != hipSuccess) return e;
  if (storage == kF16) {
    e = launch_set(EncodeField<kF16>{x, static_cast<uint16_t *>(dst), st, vf}, g, false, s);
    hipLaunchKernelGGL(scale_record_kernel<kF16>, dim3(1), dim3(64), 0, s, st, vf);
  } else {
    e = launch_set(EncodeField<kBF16>{x, static_cast<uint16_t *>(dst), st, vf}, g, false, s);
    hipLaunchKernelGGL(scale_record_kernel<kBF16>, dim3(1), dim3(64), 0, s, st, vf);
  }
  return e != hipSuccess ? e : hipGetLastError();
}

hipError_t launch_copy_in(const float *x, float *dst, const GridRows &g, hipStream_t s) {
  if (8 * g.rows * g.nx > (size_t(256) << 20)) return launch_set(CopyIn<float, 4, true>{x, dst}, g, false, s);
  return launch_set(CopyIn<float, 4>{x, dst}, g, false, s);
}

hipError_t launch_bump(StepState *st, int count, const uint32_t *slots, hipStream_t s) {
  hipLaunchKernelGGL(bump_kernel, dim3(1), dim3(64), 0, s, st, count, slots);
  return hipGetLastError();
}

hipError_t launch_set_n(StepState *st, int n, hipStream_t s) {
  hipLaunchKernelGGL(set_n_kernel, dim3(1), dim3(64), 0, s, st, n);
  return hipGetLastError();
}

hipError_t launch_noise(int storage, void *field, size_t n, uint32_t seed, hipStream_t s) {
  const dim3 g(grid_for(n, 256)), b(256);
  switch (storage) {
    case kF32: hipLaunchKernelGGL(noise_kernel<kF32>, g, b, 0, s, static_cast<float *>(field), n, seed); break;
    case kF16: hipLaunchKernelGGL(noise_kernel<kF16>, g, b, 0, s, static_cast<uint16_t *>(field), n, seed); break;
    case kBF16: hipLaunchKernelGGL(noise_kernel<kBF16>, g, b, 0, s, static_cast<uint16_t *>(field), n, seed); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_reset_state(StepState *st, uint32_t *slots, hipStream_t s) {
  hipLaunchKernelGGL(reset_state_kernel, dim3(1), dim3(64), 0, s, st, slots);
  return hipGetLastError();
}

hipError_t launch_decode(int storage, const void *field, float *out, const GridRows &g, const StepState *st,
                         int slot_off, bool v_field, hipStream_t s) {
  const int vf = v_field ? 1 : 0;
  switch (storage) {
    case kF32:
      return launch_read(Decode<kF32>{static_cast<const float *>(field), out, st, slot_off, vf}, g, false, s);
    case kF16:
      return launch_read(Decode<kF16>{static_cast<const uint16_t *>(field), out, st, slot_off, vf}, g, false, s);
    case kBF16:
      return launch_read(Decode<kBF16>{static_cast<const uint16_t *>(field), out, st, slot_off, vf}, g, false, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_decode_prev(int storage, const void *fa, const void *fv, float *out, const float *gx,
                              const float *gy, const float *gz, const GridRows &g, int ny, const StepState *st,
                              hipStream_t s) {
  const uint16_t *a = static_cast<const uint16_t *>(fa), *v = static_cast<const uint16_t *>(fv);
  const FastDiv64 dx(g.nx), dy(ny);
  if (storage == kF16) return launch_read(DecodePrev<kF16>{a, v, out, gx, gy, gz, dx, dy, FastDiv(ny), st}, g, true, s);
  if (storage == kBF16) return launch_read(DecodePrev<kBF16>{a, v, out, gx, gy, gz, dx, dy, FastDiv(ny), st}, g, true, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gather(int storage, const void *field, const int64_t *lin, int nrec, float *traces,
                         const StepState *st, int k, hipStream_t s) {
  const dim3 g((nrec + 255) / 256), b(256);
  switch (storage) {
    case kF32: hipLaunchKernelGGL(gather_kernel<kF32>, g, b, 0, s, (const float *)field, lin, nrec, traces, st, k); break;
    case kF16: hipLaunchKernelGGL(gather_kernel<kF16>, g, b, 0, s, (const uint16_t *)field, lin, nrec, traces, st, k); break;
    case kBF16: hipLaunchKernelGGL(gather_kernel<kBF16>, g, b, 0, s, (const uint16_t *)field, lin, nrec, traces, st, k); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_scatter(float *field, const int64_t *node, const int32_t *off, const int32_t *ord, int nnode,
                          int nrec, const float *m, const float *gnode, const float *resid, int row, hipStream_t s) {
  if (nnode <= 0) return hipSuccess;
  hipLaunchKernelGGL(scatter_kernel, dim3((nnode + 255) / 256), dim3(256), 0, s, field, node, off, ord, nnode, nrec, m,
                     gnode, resid, row);
  return hipGetLastError();
}

hipError_t launch_check_finite(int storage, const void *field, size_t n, StepState *st, hipStream_t s) {
  const dim3 g(grid_for(n, 256)), b(256);
  switch (storage) {
    case kF32: hipLaunchKernelGGL(finite_kernel<kF32>, g, b, 0, s, (const float *)field, n, st); break;
    case kF16: hipLaunchKernelGGL(finite_kernel<kF16>, g, b, 0, s, (const uint16_t *)field, n, st); break;
    case kBF16: hipLaunchKernelGGL(finite_kernel<kBF16>, g, b, 0, s, (const uint16_t *)field, n, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_grad_final(const float *img, const float *m, float dt, float *grad, const GridRows &g, hipStream_t s) {
  return launch_read(GradFinal{img, m, dt, grad}, g, false, s);
}

namespace {
template <int VEC>
void launch_psi(int vx, ShellWork &work, const CpmlArgs &c, const float *cur, hipStream_t s) {
  const dim3 b(256);
  work.run([&](dim3 g, const ShellWork &P) {
    if (vx == 4) hipLaunchKernelGGL((cpml_psi_kernel<VEC, 4>), g, b, 0, s, c, P, cur);
    else if (vx == 2) hipLaunchKernelGGL((cpml_psi_kernel<VEC, 2>), g, b, 0, s, c, P, cur);
    else hipLaunchKernelGGL((cpml_psi_kernel<VEC, 1>), g, b, 0, s, c, P, cur);
  });
}
// x nodes per lane: as many of 4, 2, 1 as divide every length given
int lane_width(int a, int b) { return a % 4 == 0 && b % 4 == 0 ? 4 : (a % 2 == 0 && b % 2 == 0 ? 2 : 1); }
}  // namespace

hipError_t launch_cpml_psi(const CpmlArgs &c, const float *cur, hipStream_t s) {
  const int vec = lane_width(c.nx, 4), vx = lane_width(c.nx, c.W);
  ShellWork P(c, c.W, vx);
  if (vec == 4) launch_psi<4>(vx, P, c, cur, s);
  else if (vec == 2) launch_psi<2>(vx, P, c, cur, s);
  else launch_psi<1>(vx, P, c, cur, s);
  return hipGetLastError();
}

hipError_t launch_cpml_fix(const CpmlArgs &c, const float *cur, const float *m, float *out, bool yz_only,
                           hipStream_t s) {
  const Shell S(c.W + kRadius, c.nx, c.ny, c.nz);
  if (yz_only) {
    const int vec = lane_width(c.nx, 4);
    ShellWork work(c, c.W + kRadius, 0, kFixRows);
    const dim3 b(256);
    work.run([&](dim3 g, const ShellWork &P) {
      if (vec == 4) hipLaunchKernelGGL(cpml_fix_yz_kernel<4>, g, b, 0, s, c, P, cur, m, out);
      else if (vec == 2) hipLaunchKernelGGL(cpml_fix_yz_kernel<2>, g, b, 0, s, c, P, cur, m, out);
      else hipLaunchKernelGGL(cpml_fix_yz_kernel<1>, g, b, 0, s, c, P, cur, m, out);
    });
    return hipGetLastError();
  }
  const unsigned n = S.count();
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(cpml_fix_kernel, dim3((n + 255) / 256), dim3(256), 0, s, c, cur, m, out);
  return hipGetLastError();
}

namespace {
template <typename V> hipError_t copy_rows(V *snap, V *field, const GridRows &g, bool save, hipStream_t s) {
  return save ? launch_read(CopyOut<V, 1>{field, snap}, g, false, s) : launch_set(CopyIn<V, 1>{snap, field}, g, false, s);
}
}  // namespace

hipError_t launch_copy_rows(int storage, void *snap, void *field, const GridRows &g, bool save, hipStream_t s) {
  if (storage == kF32) return copy_rows(static_cast<uint32_t *>(snap), static_cast<uint32_t *>(field), g, save, s);
  return copy_rows(static_cast<uint16_t *>(snap), static_cast<uint16_t *>(field), g, save, s);
}

hipError_t launch_fill_zero(void *p, size_t bytes, hipStream_t s) {
  const size_t n16 = bytes / 16;
  const size_t tail = bytes - n16 * 16;
  hipLaunchKernelGGL(zero_kernel, dim3(grid_for(n16 ? n16 : 1, 256)), dim3(256), 0, s, static_cast<uint4 *>(p), n16,
                     static_cast<uint8_t *>(p) + n16 * 16, tail);
  return hipGetLastError();
}

}  // namespace wave
