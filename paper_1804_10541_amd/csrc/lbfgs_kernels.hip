// Kernels of the L-BFGS initial-matrix solve (Sec. 2.3.2):
// x = H_0^{-1} v with H_0 = 2 alpha hbar^y L^T L + gamma I (curvature) or
// -alpha hbar^y L + gamma I (diffusive regulariser).
//
// The 7-point Laplacian with clamped (Neumann) neighbours is the Kronecker sum
// of one-dimensional second-difference matrices whose eigenvectors are the
// DCT-II cosines, so H_0 is diagonal in the separable cosine basis: the solve
// is a forward transform along z, y and x, a division by the eigenvalues
// 2 alpha hbar^y (lx + ly + lz)^2 + gamma (curvature) or
// -alpha hbar^y (lx + ly + lz) + gamma (diffusive), and the inverse transform.
//
// Each axis transform is a dense product of the orthonormal cosine matrix C
// (n x n) with all lines of that axis.  C[k][n-1-i] = (-1)^k C[k][i], so with
// H = ceil(n/2), e_i = x_i + x_{n-1-i} and o_i = x_i - x_{n-1-i} (i < H) the even
// and the odd outputs are two products of H x H matrices with e and o: half the
// operations.  They run on the matrix cores in float32 (v_mfma_f32_16x16x4:
// float32 products and sums, as the vector units form them).
#include <algorithm>

#include "mfr_internal.h"

namespace mfr {

namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int TL = 64;      // lines per work-group (16 per wave)
constexpr int KC = 16;      // summed entries per chunk
constexpr int AP = KC + 4;  // pitches in LDS: 16-byte reads of 8 rows on distinct banks
constexpr int BP = TL + 4;
constexpr int kRowTiles = kH0Half / 16;   // most row tiles of a group

// Lines of an axis: line l < lines starts at (l / C) bs + (l % C) cs, its entries
// are `is` apart.
struct Lines {
  int n, H;
  long long bs, is, cs, lines;
  int C;
  __device__ __forceinline__ long long base(long long l) const { return (l / C) * bs + (l % C) * cs; }
};

struct ScaleArgs {
  const float* lam;   // eigenvalues along x, y, z
  int nx, ny, nz;
  float c2, c1, gamma;
};

enum AxisMode : int { FWD = 0, INV = 1, MID = 2 };

// FWD, INV: out = C in, C^T in along an axis whose lines lie side by side (y, z).
// MID: the x axis, whose entries are contiguous: forward transform, division by the
// eigenvalues and inverse transform of 64 lines without leaving the registers: the
// accumulators of the first product (row 4 quad + r in register r) are the second
// one's operands for the summed entries 4 quad + r.
// A: the even H x H matrix, then the odd one (rows outputs, columns inputs); G: the
// same of the inverse (MID).  NRT: row tiles of 16 output pairs per group.
//
// Bound by the matrix cores (16 of a tile's rows and lines per instruction; 129
// nodes take 80 rows for 65) and the passes over the vector (18 us each at
// 129x129x225 nodes, three components; times at launch_h0_solve).
template <int NRT, int MODE>
__global__ __launch_bounds__(256) void axis_kernel(const Lines L, const float* __restrict__ A,
                                                   const float* __restrict__ G, const float* __restrict__ in,
                                                   float* __restrict__ out, const ScaleArgs sc) {
  __shared__ __align__(16) float sA[2][NRT * 16][AP];
  __shared__ float sB[2][KC][BP];
  constexpr bool I1 = MODE == MID;   // the summed index is the contiguous one
  const int tid = threadIdx.x, lane = tid & 63, c16 = lane & 15, quad = lane >> 4, wave = tid >> 6;
  const int n = L.n, H = L.H;
  const int row0 = blockIdx.y * NRT * 16;
  const long long l0 = (long long)blockIdx.x * TL;

  // this thread's entries of a chunk: strided lines: line tid % 64, entries tid / 64
  // + 4 j; contiguous ones: entry tid % 16, lines tid / 16 + 16 j
  long long lb[4];
  bool lv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const long long l = l0 + (I1 ? (tid >> 4) + 16 * j : tid & 63);
    lv[j] = l < L.lines;
    if (I1 || j == 0) lb[j] = L.base(lv[j] ? l : 0);
  }
  float pa[2][NRT], pe[4], po[4];
  auto load_a = [&](const float* __restrict__ M, int i0) {
    const int k = i0 + (tid & 15);
#pragma unroll
    for (int j = 0; j < NRT; ++j) {
      const int row = row0 + (tid >> 4) + 16 * j;
      const bool ok = row < H && k < H;
#pragma unroll
      for (int p = 0; p < 2; ++p) pa[p][j] = ok ? M[((size_t)p * H + row) * H + k] : 0.0f;
    }
  };
  auto load_b = [&](int i0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = i0 + (I1 ? tid & 15 : (tid >> 6) + 4 * j);
      const float* const p = in + (I1 ? lb[j] : lb[0]);
      const bool v = I1 ? lv[j] : lv[0];
      if constexpr (MODE == INV) {   // even and odd coefficients
        pe[j] = v && 2 * i < n ? p[2 * (long long)i * L.is] : 0.0f;
        po[j] = v && 2 * i + 1 < n ? p[(2 * (long long)i + 1) * L.is] : 0.0f;
      } else {
        const bool ok = v && i < H;
        const float a = ok ? p[(long long)i * (I1 ? 1 : L.is)] : 0.0f;
        const float b = ok && n - 1 - i != i ? p[(long long)(n - 1 - i) * (I1 ? 1 : L.is)] : 0.0f;
        pe[j] = a + b;
        po[j] = n - 1 - i != i ? a - b : 0.0f;   // (the middle entry of an odd n has no odd part)
      }
    }
  };
  auto store_a = [&]() {
#pragma unroll
    for (int j = 0; j < NRT; ++j)
#pragma unroll
      for (int p = 0; p < 2; ++p) sA[p][(tid >> 4) + 16 * j][tid & 15] = pa[p][j];
  };
  auto store_b = [&]() {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int k = I1 ? tid & 15 : (tid >> 6) + 4 * j, l = I1 ? (tid >> 4) + 16 * j : tid & 63;
      sB[0][k][l] = pe[j];
      sB[1][k][l] = po[j];
    }
  };
  // acc[p][rt] += A rows x (be, bo): the summed entry of quad q in step s is 4 q + s
  auto mul = [&](f32x4 (&acc)[2][NRT], const f32x4 be, const f32x4 bo) {
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
      const f32x4 ae = *reinterpret_cast<const f32x4*>(&sA[0][rt * 16 + c16][4 * quad]);
      const f32x4 ao = *reinterpret_cast<const f32x4*>(&sA[1][rt * 16 + c16][4 * quad]);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        acc[0][rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ae[s], be[s], acc[0][rt], 0, 0, 0);
        acc[1][rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(ao[s], bo[s], acc[1][rt], 0, 0, 0);
      }
    }
  };

  f32x4 acc[2][NRT];
#pragma unroll
  for (int rt = 0; rt < NRT; ++rt) acc[0][rt] = acc[1][rt] = (f32x4){0.f, 0.f, 0.f, 0.f};
  load_a(A, 0);
  load_b(0);
  for (int i0 = 0; i0 < H; i0 += KC) {
    store_a();
    store_b();
    __syncthreads();
    if (i0 + KC < H) {
      load_a(A, i0 + KC);
      load_b(i0 + KC);
    } else if constexpr (MODE == MID) {
      load_a(G, 0);
    }
    f32x4 be, bo;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      be[s] = sB[0][4 * quad + s][16 * wave + c16];
      bo[s] = sB[1][4 * quad + s][16 * wave + c16];
    }
    mul(acc, be, bo);
    __syncthreads();
  }

  const long long line = l0 + 16 * wave + c16;
  if constexpr (MODE != MID) {
    if (line >= L.lines) return;
    float* const p = out + L.base(line);
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = row0 + rt * 16 + 4 * quad + r;
        const float e = acc[0][rt][r], o = acc[1][rt][r];
        if constexpr (MODE == FWD) {
          if (2 * row < n) p[2 * (long long)row * L.is] = e;
          if (2 * row + 1 < n) p[(2 * (long long)row + 1) * L.is] = o;
        } else {
          if (row >= H) continue;
          p[(long long)row * L.is] = e + o;
          if (n - 1 - row != row) p[(long long)(n - 1 - row) * L.is] = e - o;
        }
      }
  } else {
    // the division in the cosine basis
    const long long lc = min(line, L.lines - 1);
    const float ly = sc.lam[sc.nx + (int)(lc % sc.ny)];
    const float lz = sc.lam[sc.nx + sc.ny + (int)((lc / sc.ny) % sc.nz)];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int k = 2 * (rt * 16 + 4 * quad + r) + p;
          const float l = sc.lam[min(k, n - 1)] + ly + lz;
          acc[p][rt][r] = k < n ? acc[p][rt][r] / fmaf(fmaf(sc.c2, l, sc.c1), l, sc.gamma) : 0.0f;
        }
    f32x4 res[2][NRT];
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) res[0][rt] = res[1][rt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kt = 0; kt < NRT; ++kt) {
      store_a();
      __syncthreads();
      if (kt + 1 < NRT) load_a(G, (kt + 1) * KC);
      mul(res, acc[0][kt], acc[1][kt]);
      __syncthreads();
    }
    // through LDS, so that the stores run along the lines: entries i and n-1-i
    static_assert(TL * 33 <= 2 * KC * BP, "the staging fits sB");
    float* const st = &sB[0][0][0];   // [TL][33]
#pragma unroll
    for (int rt = 0; rt < NRT; ++rt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float e = res[0][rt][r], o = res[1][rt][r];
        st[(16 * wave + c16) * 33 + 4 * quad + r] = e + o;
        st[(16 * wave + c16) * 33 + 16 + 4 * quad + r] = e - o;
      }
      __syncthreads();
      const int i = rt * 16 + (tid & 15);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int l = (tid >> 4) + 16 * j;
        if (lv[j] && i < H) {
          float* const p = out + lb[j];
          p[i] = st[l * 33 + (tid & 15)];
          if (n - 1 - i != i) p[n - 1 - i] = st[l * 33 + 16 + (tid & 15)];
        }
      }
      __syncthreads();
    }
  }
}

// ---- x axes of more than 2 kH0Half nodes ------------------------------------------
constexpr int TK = 32;   // output rows (transformed index) per tile
constexpr int TC = 64;   // lines per tile
constexpr int TI = 32;   // summation chunk

// out[c][k] = sum_i M[k][i] in[c][i] for C contiguous lines of n entries.
__global__ __launch_bounds__(256) void long_axis_kernel(const float* __restrict__ M, int n, const float* __restrict__ in,
                                                        float* __restrict__ out, int C) {
  __shared__ float sM[TK][TI + 1];
  __shared__ float sIn[TI][TC + 4];
  const int tid = threadIdx.x;
  const int c0 = blockIdx.x * TC, k0 = blockIdx.y * TK;
  const int tk = tid / 16, tc = tid % 16;   // rows 2 tk, 2 tk + 1; columns 4 tc .. 4 tc + 3
  float acc[2][4] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  for (int i0 = 0; i0 < n; i0 += TI) {
    for (int e = tid; e < TK * TI; e += 256) {
      const int kk = e / TI, ii = e % TI;
      const int k = k0 + kk, i = i0 + ii;
      sM[kk][ii] = (k < n && i < n) ? M[(size_t)k * n + i] : 0.0f;
    }
    for (int e = tid; e < TI * TC; e += 256) {
      const int ii = e % TI, cc = e / TI;
      const int i = i0 + ii, c = c0 + cc;
      sIn[ii][cc] = (i < n && c < C) ? in[(long long)c * n + i] : 0.0f;
    }
    __syncthreads();
#pragma unroll 8
    for (int ii = 0; ii < TI; ++ii) {
      const float m0 = sM[2 * tk][ii], m1 = sM[2 * tk + 1][ii];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float v = sIn[ii][4 * tc + j];
        acc[0][j] = fmaf(m0, v, acc[0][j]);
        acc[1][j] = fmaf(m1, v, acc[1][j]);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int k = k0 + 2 * tk + r;
    if (k >= n) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int c = c0 + 4 * tc + j;
      if (c < C) out[(long long)c * n + k] = acc[r][j];
    }
  }
}

// x = v / (c2 l^2 + c1 l + gamma), l = lx[i] + ly[j] + lz[k], in the cosine basis.
__global__ __launch_bounds__(256) void h0_scale_kernel(float* __restrict__ x, const ScaleArgs s, int nc) {
  const size_t nb = (size_t)s.nx * s.ny * s.nz, total = (size_t)nc * nb;
  const float* lx = s.lam;
  const float* ly = s.lam + s.nx;
  const float* lz = s.lam + s.nx + s.ny;
  for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += (size_t)gridDim.x * blockDim.x) {
    const size_t n = idx % nb;
    const int i = (int)(n % s.nx), j = (int)((n / s.nx) % s.ny), k = (int)(n / ((size_t)s.nx * s.ny));
    const float l = lx[i] + ly[j] + lz[k];
    x[idx] = x[idx] / fmaf(fmaf(s.c2, l, s.c1), l, s.gamma);
  }
}

// ---- the tables ---------------------------------------------------------------------
struct TableArgs {
  int n[3];
  double hy[3];
  int full;   // the x axis takes the whole matrices
  float* C[3];
  float* Ct[3];
  float* lam;
};

// Cosine tables of one axis (blockIdx.y), formed in float64 from exactly reduced
// arguments: C the forward matrices [parity][k'][i] = C[2 k' + parity][i] (H x H
// each), Ct the same transposed; the whole n x n matrices where the axis is long;
// and the eigenvalues -4 sin^2(pi k / 2n) / hy^2.
__global__ __launch_bounds__(256) void h0_table_kernel(const TableArgs t) {
  const int d = blockIdx.y, n = t.n[d], H = (n + 1) / 2;
  const bool full = d == 0 && t.full;
  int off = 0;
  for (int e = 0; e < d; ++e) off += t.n[e];
  const size_t entries = full ? (size_t)n * n : 2 * (size_t)H * H;
  for (size_t q = (size_t)blockIdx.x * 256 + threadIdx.x; q < entries; q += (size_t)gridDim.x * 256) {
    int k, i;
    size_t tr;   // the entry's place in the transposed table
    if (full) {
      k = (int)(q / n);
      i = (int)(q % n);
      tr = (size_t)i * n + k;
    } else {
      const int p = (int)(q / ((size_t)H * H));
      const size_t r = q - (size_t)p * H * H;
      const int kk = (int)(r / H);
      i = (int)(r % H);
      k = 2 * kk + p;
      tr = ((size_t)p * H + i) * H + kk;
    }
    float v = 0.0f;
    if (k < n) {
      const long long m = (long long)k * (2 * i + 1) % (4LL * n);   // cos(pi m / 2n) has period 4n
      // the middle entry of an odd length is a zero of the odd cosines
      if (!((k & 1) && 2 * i + 1 == n)) v = (float)(sqrt((k == 0 ? 1.0 : 2.0) / n) * cospi((double)m / (2.0 * n)));
    }
    t.C[d][q] = v;
    t.Ct[d][tr] = v;
  }
  if (blockIdx.x == 0)
    for (int k = threadIdx.x; k < n; k += 256) {
      const double s = sinpi(k / (2.0 * n));
      t.lam[off + k] = (float)(-4.0 * s * s / (t.hy[d] * t.hy[d]));
    }
}

template <int MODE>
hipError_t launch_axis(const Lines& L, const float* A, const float* G, const float* in, float* out, const ScaleArgs& sc,
                       hipStream_t st) {
  const int tiles = (L.H + 15) / 16, nrt = std::min(tiles, kRowTiles);
  const dim3 grid((unsigned)((L.lines + TL - 1) / TL), (unsigned)((tiles + nrt - 1) / nrt));
  switch (nrt) {
    case 1: hipLaunchKernelGGL((axis_kernel<1, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
    case 2: hipLaunchKernelGGL((axis_kernel<2, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
    case 3: hipLaunchKernelGGL((axis_kernel<3, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
    case 4: hipLaunchKernelGGL((axis_kernel<4, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
    case 5: hipLaunchKernelGGL((axis_kernel<5, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
    case 6: hipLaunchKernelGGL((axis_kernel<6, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
    case 7: hipLaunchKernelGGL((axis_kernel<7, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
    default: hipLaunchKernelGGL((axis_kernel<8, MODE>), grid, dim3(256), 0, st, L, A, G, in, out, sc); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_h0_tables(const H0Tables& t, const double hy[3], hipStream_t st) {
  TableArgs a{};
  size_t most = 1;
  for (int d = 0; d < 3; ++d) {
    a.n[d] = t.n[d];
    a.hy[d] = hy[d];
    a.C[d] = const_cast<float*>(t.C[d]);
    a.Ct[d] = const_cast<float*>(t.Ct[d]);
    most = std::max(most, (size_t)t.n[d] * t.n[d]);
  }
  a.full = t.n[0] > 2 * kH0Half;
  a.lam = const_cast<float*>(t.lam);
  const unsigned blocks = (unsigned)std::min<size_t>((most + 255) / 256, 1024);
  hipLaunchKernelGGL(h0_table_kernel, dim3(blocks, t.n[2] > 1 ? 3 : 2), dim3(256), 0, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || t.n[2] > 1) return e;
  return launch_fill(1, 0.0f, a.lam + t.n[0] + t.n[1], st);   // (no z transform: eigenvalue 0)
}

// x = H_0^{-1} v.  ta, tb: scratch node vectors; x may alias v.
// Five passes over the vector (z, y, x there and back, y, z), each read and written
// once, against seven with a float32 product per axis and direction on the vector
// units and the division apart.  A call at 129x129x225 nodes, three components 1024 ->
// 290 us; its kernels in a trace (which runs them a little slower): z 175 + 175 -> 65 +
// 60 us, y 175 + 175 -> 42 + 40 us, x with the division 138 + 36 + 138 -> 87 us; tables:
// seven copies from the host -> 5 us.
// An x axis of more than 2 kH0Half nodes, whose 64 lines do not fit the registers,
// takes the whole matrices and the division apart: 257x33x33 nodes 205 -> 128 us (256:
// 201 -> 69 us), 513x129x65 nodes 1423 -> 1010 us.
hipError_t launch_h0_solve(const H0Tables& t, const float* v, float* x, float* ta, float* tb, float c2, float c1,
                           float gamma, hipStream_t st) {
  const int nx = t.n[0], ny = t.n[1], nz = t.n[2], nc = t.nc;
  const long long nxy = (long long)nx * ny, nb = nxy * nz;
  const ScaleArgs sc{t.lam, nx, ny, nz, c2, c1, gamma};
  const Lines Lz{nz, (nz + 1) / 2, nb, nxy, 1, nc * nxy, (int)nxy};
  const Lines Ly{ny, (ny + 1) / 2, nxy, nx, 1, (long long)nc * nz * nx, nx};
  const Lines Lx{nx, (nx + 1) / 2, 0, 1, nx, (long long)nc * nz * ny, (int)((long long)nc * nz * ny)};
  hipError_t e;
  const float* in = v;
  if (nz > 1) {   // a two-dimensional field has no z transform
    if ((e = launch_axis<FWD>(Lz, t.C[2], nullptr, v, tb, sc, st)) != hipSuccess) return e;
    in = tb;
  }
  if ((e = launch_axis<FWD>(Ly, t.C[1], nullptr, in, ta, sc, st)) != hipSuccess) return e;
  float* mid = tb;
  if (nx <= 2 * kH0Half) {
    if ((e = launch_axis<MID>(Lx, t.C[0], t.Ct[0], ta, tb, sc, st)) != hipSuccess) return e;
  } else {
    const int C = (int)Lx.lines;
    const dim3 grid((C + TC - 1) / TC, (nx + TK - 1) / TK);
    hipLaunchKernelGGL(long_axis_kernel, grid, dim3(256), 0, st, t.C[0], nx, ta, tb, C);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const int blocks = (int)std::min<long long>((nc * nb + 255) / 256, 8192);
    hipLaunchKernelGGL(h0_scale_kernel, dim3(blocks), dim3(256), 0, st, tb, sc, nc);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(long_axis_kernel, grid, dim3(256), 0, st, t.Ct[0], nx, tb, ta, C);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    mid = ta;
  }
  if (nz == 1) return launch_axis<INV>(Ly, t.Ct[1], nullptr, mid, x, sc, st);
  float* const back = mid == tb ? ta : tb;
  if ((e = launch_axis<INV>(Ly, t.Ct[1], nullptr, mid, back, sc, st)) != hipSuccess) return e;
  return launch_axis<INV>(Lz, t.Ct[2], nullptr, back, x, sc, st);
}

}  // namespace mfr
