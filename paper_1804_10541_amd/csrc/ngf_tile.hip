// Fused matrix-free NGF kernel on voxel tiles (CDNA4 / gfx950).
//
// One work-group covers a column block of BX x BY voxel columns: it owns the
// rows of dr at the inner (BX-2) x (BY-2) columns and samples the template on
// a one-column ring around them as well, which the differences of its rows
// need.  The group marches through a chunk of z planes; each thread owns one
// column and keeps the values of its own column in registers across planes,
// while the x/y neighbours of the current plane are exchanged through LDS.
// Per step t three stages run:
//
//  A(t)   conversion P of u (and of p) at plane t (Sec. 4.3,
//         eq. grid_conversion), trilinear template sample T(hat-y) and its
//         derivative g = dT/dP (eq. dT), and, for the Hessian product,
//         a = g . (P p);
//  B(t-1) the six short differences of T(P y) and R (eq. gradient_discretized
//         with clamped neighbours, eq. boundary_conditions), the residual r
//         (eq. residual) and the row rho-hat of dr (eq. rho, eq. hatRho);
//         then z_l = (dr a)_l (Hessian) or z_l = r_l (gradient) and the
//         products e_l(k) = rho-hat_l(k) z_l;
//  C(t-2) the column sum w_i = sum_{rows l} dr_{l,i} z_l = e_i(0) +
//         sum_k e_{i+k}(-k) over neighbours inside the image (eq. gradNGF and
//         eq. drTdr / eq. hessMult as a gather over the rows of dr), v = g w,
//         accumulated into the node planes of the transposed conversion P^T.
//         A group gathers only its own rows, at every column it covers (own
//         columns and ring): a ring column is an own column of the
//         neighbouring group, which adds the contributions of its rows there,
//         and P^T is linear, so the two partial node blocks sum to the whole.
//         Each row's contributions are formed exactly once.
//
// Columns and planes outside the image sample the template at the clamped
// position, so every neighbour read in stage B already holds the clamped
// value of eq. boundary_conditions (differences across the border are 0).
// The stage-A inputs of plane t+1 (template corners, reference value) are
// loaded during step t.  The march is unrolled by three so the per-column
// register windows (planes t, t-1, t-2) sit in fixed registers.
//
// P^T is a gather: each column accumulates its z contributions in registers;
// when a node plane is complete the group reduces it over x and y on the matrix
// cores and writes the node block to its own slot of a partial buffer.  A node pass sums
// the slots that overlap each node in a fixed order, so results are
// deterministic and no atomics are used.  Nothing per voxel reaches HBM.
//
// The same march evaluates the sum-of-squared-differences distance (SSD,
// Sec. 4.4), whose residual Jacobian dr/dT is the identity: stage B forms
// r = T(P y) - R and z_l = a_l (Hessian) or r_l (gradient) at the own columns,
// stage C takes w_i = z_i, and no plane data is exchanged through LDS.
#include <type_traits>

#include "tile_common.h"

namespace mfr {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// LDS of one work-group of the voxel-tile kernel.
template <int BX, int BY, int MODE, bool SSD>
struct TileSmem {
  static constexpr int NT = BX * BY, MAXNX = BX + 1, MAXNY = BY + 1;
  static constexpr bool HV = (MODE == MODE_HV), NEED_C = (MODE != MODE_OBJ);
  static constexpr int NX = SSD ? 1 : NT;   // plane exchange (NGF differences only)
  // with a zero pad of one block row at both ends, so that every lane's four
  // neighbour reads stay inside the arrays and read finite values
  static constexpr int XP = SSD ? 0 : BX;
  float sTw[2][NX + 2 * XP];
  float sR[2][NX + 2 * XP];
  float sA[HV ? 2 : 1][HV ? NX + 2 * XP : 1];
  // row products of the plane exchange, with a zero pad of one block row at both
  // ends: a neighbour read past the block's edge (or wrapping to the next row,
  // whose edge column is a ring column that writes 0) then adds exactly 0
  static constexpr int EP = (NEED_C && !SSD) ? BX : 0;
  float sE[NEED_C ? 2 : 1][4][NEED_C ? NX + 2 * EP : 1];
  // a finished node plane of P^T, per column, waiting for its reduction over x and
  // y; the pitch spreads the rows over the banks
  static constexpr int VP = BX + 4;
  float sV[NEED_C ? 3 : 1][NEED_C ? BY * VP : 1];
  // conversion weights as the operands of that reduction: [node tile][step][lane]
  static constexpr int XT = (MAXNX + 15) / 16, YT = (MAXNY + 15) / 16, RT = (BY + 15) / 16;
  float sWx[NEED_C ? XT : 1][NEED_C ? BX / 4 : 1][NEED_C ? 64 : 1];
  float sWy[NEED_C ? YT : 1][NEED_C ? 4 * RT : 1][NEED_C ? 64 : 1];
  Conv1 sCx[BX], sCy[BY];
  // u and p of the own column at the upper one of the two node planes in use (own
  // slot only): read when the march passes to the next node plane, not kept in registers
  float sHi[HV ? 6 : 3][NT];
  // Node values of the block, one node plane ahead of the march (u's, then p's), and
  // where this thread's two of a component set lie in a node plane.  Not for SSD, whose
  // steps hold no barrier, nor where a CU would lose its second group (the LDS of 64 x 8
  // columns) or registers spill (the gradient of 1024 columns).
  static constexpr bool STG = !SSD && (NT > 512 ? HV : BX == 32);
  float sN[HV ? 2 : 1][STG ? 2 * NT : 1];
  unsigned sSrc[2][STG ? NT : 1];
  // z conversion and template-coordinate entries of planes zb-2 .. ze+1 (clamped
  // into the image): read at a uniform index every plane, from LDS rather than
  // through a vector load whose latency would sit on every step's address path
  Conv1 sCz[kMaxChunk + 4];
  Samp1 sSz[kMaxChunk + 4];
  double sRed[NT / 64];
};

// One tile (work-group id `bid` of the problem P) of the fused kernel.
template <int BX, int BY, int MODE, bool SSD>
__device__ __forceinline__ void tile_body(const TileParams& P, const int bid, const float* __restrict__ u,
                                          const float* __restrict__ pv, TileSmem<BX, BY, MODE, SSD>& S) {
  constexpr int NT = BX * BY;
  constexpr int TX = BX - 2, TY = BY - 2;   // own columns per tile
  constexpr bool HV = (MODE == MODE_HV);
  constexpr bool NEED_C = (MODE != MODE_OBJ);
  auto& sTw = S.sTw;
  auto& sR = S.sR;
  auto& sA = S.sA;
  auto& sE = S.sE;
  using Sm = TileSmem<BX, BY, MODE, SSD>;
  constexpr int EP = Sm::EP, VP = Sm::VP;
  auto& sV = S.sV;
  auto& sWx = S.sWx;
  auto& sWy = S.sWy;
  auto& sCx = S.sCx;
  auto& sCy = S.sCy;
  auto& sCz = S.sCz;
  auto& sSz = S.sSz;
  auto& sRed = S.sRed;

  const int tid = threadIdx.x;
  const int tx = tid % BX, ty = tid / BX;

  const int tile_x = bid % P.tiles_x;
  const int rest = bid / P.tiles_x;
  const int tile_y = rest % P.tiles_y;
  const int chunk = rest / P.tiles_y;
  const int x0 = tile_x * TX, y0 = tile_y * TY;
  const int zb = chunk * P.chunk_len;
  const int ze = min(P.mz, zb + P.chunk_len);

  // Columns: the own columns tx in [1, BX-2] plus a one-column ring.  Stage B
  // forms the rows of dr at own columns only; stage C gathers, at every column
  // of the group inside the image, the contributions of the group's own rows
  // (the ring's other contributions come from the neighbouring group, whose
  // own columns they are) and the transposed conversion sums both groups'
  // partial node blocks.
  const int gx = x0 - 1 + tx, gy = y0 - 1 + ty;
  const bool in_img = (gx >= 0) && (gx < P.mx) && (gy >= 0) && (gy < P.my);
  const bool own = (tx >= 1) && (tx < BX - 1) && (ty >= 1) && (ty < BY - 1);
  const bool inB = own && in_img;
  const bool inC = in_img;
  const float own_row = inB ? 1.0f : 0.0f;   // scales z_l: 0 for rows this group does not own

  // own column, clamped into the image
  const int cxi = min(max(gx, 0), P.mx - 1), cyi = min(max(gy, 0), P.my - 1);
  const Samp1 spx = P.sx[cxi], spy = P.sy[cyi];
  // Template cells are counted from the padded template's first one (cell -2); its byte
  // pitches, which a 24-bit multiply (full rate) takes where they fit.
  const int bx2 = spx.base + 2, by2 = spy.base + 2;
  const unsigned px4 = 4u * (unsigned)P.PX, pxy4 = 4u * (unsigned)P.PXY;
  const bool mul24 = pxy4 < (1u << 24) && px4 < (1u << 24);
  const unsigned nxy = (unsigned)(P.nx * P.ny);
  const unsigned plane = (unsigned)(P.mx * P.my);
  const unsigned colxy = (unsigned)(cyi * P.mx + cxi);
  const unsigned nb = (unsigned)P.nbar, nxu = (unsigned)P.nx;

  // Local columns [lxa, lxb] and rows [lya, lyb] of the group inside the image,
  // the first node they touch and the number of node columns / rows touched.
  const int lxa = x0 == 0 ? 1 : 0, lya = y0 == 0 ? 1 : 0;
  const int lxb = min(BX - 1, P.mx - x0), lyb = min(BY - 1, P.my - y0);
  const int nox = P.cx[x0 - 1 + lxa].n0, noy = P.cy[y0 - 1 + lya].n0, noz = P.cz[zb].n0;
  for (int j = tid; j < ze - zb + 4; j += NT) {
    const int q = min(max(zb - 2 + j, 0), P.mz - 1);
    sCz[j] = P.cz[q];
    Samp1 e = P.sz[q];
    e.base += 2;   // counted from the padded template's first plane
    sSz[j] = e;
  }
  if (tid < BX) sCx[tid] = P.cx[min(max(x0 - 1 + tid, 0), P.mx - 1)];
  if (tid < BY) sCy[tid] = P.cy[min(max(y0 - 1 + tid, 0), P.my - 1)];
  __syncthreads();
  constexpr int XP = TileSmem<BX, BY, MODE, SSD>::XP;
  if constexpr (XP > 0) {   // nor are the pads of the plane exchange
    for (int w = tid; w < 2 * 2 * XP; w += NT) {
      const int r = w % (2 * XP), sl = w / (2 * XP);
      const int q = r < XP ? r : NT + r;
      sTw[sl][q] = 0.f;
      sR[sl][q] = 0.f;
      if constexpr (HV) sA[sl][q] = 0.f;
    }
  }
  if constexpr (EP > 0) {   // the pads of sE are never written by the march
    for (int w = tid; w < 2 * 4 * 2 * EP; w += NT) {
      const int r = w % (2 * EP), k = (w / (2 * EP)) % 4, sl = w / (8 * EP);
      sE[sl][k][r < EP ? r : NT + r] = 0.f;
    }
  }
  const int nxl = P.cx[x0 - 1 + lxb].n0 + 2 - nox;
  const int nyl = P.cy[y0 - 1 + lyb].n0 + 2 - noy;
  if constexpr (NEED_C) {
    for (int w = tid; w < ((nxl + 15) / 16) * (BX / 4) * 64; w += NT) {
      const int c16 = w & 15, l = (w >> 4) % BX, nt = w / (16 * BX);   // lane (l & 3, c16) of step l / 4
      sWx[nt][l >> 2][w & 63] = conv_weight(sCx[l], nox + 16 * nt + c16);
    }
    for (int w = tid; w < ((nyl + 15) / 16) * Sm::RT * 256; w += NT) {
      const int lane = w & 63, r = (w >> 6) % (4 * Sm::RT), mt = w / (256 * Sm::RT);
      const int row = (r >> 2) * 16 + 4 * (lane >> 4) + (r & 3);
      sWy[mt][r][lane] = row < BY ? conv_weight(sCy[min(row, BY - 1)], noy + 16 * mt + (lane & 15)) : 0.f;
    }
  }

  // the group's partial slot: node n of component d at part[d nbar + n], n the
  // node's index in the grid, so the node pass reads its slots coalesced
  const int pslot = ((chunk % P.smz) * P.smy + tile_y % P.smy) * P.smx + tile_x % P.smx;
  float* const part = P.part + (size_t)pslot * 3 * (size_t)P.nbar;

  // Reduction of component d of the node plane in sV (local index kloc) over x,
  // then y, for the 16 node columns from 16 nt on, by one wave: two products with
  // the conversion weights on the matrix cores (v_mfma_f32_16x16x4: float32
  // products and sums).  The first leaves D[row][node x] with row 4 quad + r in
  // register r, which is what the second takes as its operand for the rows 4 quad
  // + r, so nothing goes through LDS in between: 12 matrix instructions per
  // component for up to 16 x 16 nodes.
  auto reduce = [&](int kloc, int d, int nt) {
    if constexpr (NEED_C) {
      constexpr int RT = Sm::RT, KS = BX / 4, G = RT > 1 ? 4 : 8;   // row tiles, steps, steps per load group
      // (opaque here, so that nothing of the reduction is kept in registers over the march)
      int lane = tid & 63;
      asm volatile("" : "+v"(lane));
      const int c16 = lane & 15, quad = lane >> 4;
      const float* const V = &sV[d][0];
      const size_t o0 = (size_t)d * P.nbar + (size_t)(noz + kloc) * nxy + (size_t)noy * P.nx + nox;
      f32x4 acc[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float* const row = V + min(rt * 16 + c16, BY - 1) * VP + quad;
        f32x4 s0 = (f32x4){0.f, 0.f, 0.f, 0.f}, s1 = s0;   // two chains: half the latency
#pragma unroll
        for (int i = 0; i < KS; i += G) {
          if constexpr (RT > 1) __builtin_amdgcn_sched_barrier(0);   // (registers)
          float a[G], b[G];
#pragma unroll
          for (int j = 0; j < G; ++j) {
            a[j] = row[4 * (i + j)];
            b[j] = sWx[nt][i + j][lane];
          }
#pragma unroll
          for (int j = 0; j < G; j += 2) {
            s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j + 1], b[j + 1], s1, 0, 0, 0);
          }
        }
        acc[rt] = s0 + s1;
      }
#pragma clang loop unroll(disable)
      for (int mt = 0; mt * 16 < nyl; ++mt) {
        f32x4 o = (f32x4){0.f, 0.f, 0.f, 0.f}, o1 = o;
        {
          float a[4 * RT];
#pragma unroll
          for (int r = 0; r < 4 * RT; ++r) a[r] = sWy[mt][r][lane];
#pragma unroll
          for (int r = 0; r < 4 * RT; r += 2) {
            o = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], acc[r >> 2][r & 3], o, 0, 0, 0);
            o1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r + 1], acc[r >> 2][(r & 3) + 1], o1, 0, 0, 0);
          }
          o += o1;
        }
        auto store = [&]() {
          if (16 * nt + c16 < nxl) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int fr = 16 * mt + 4 * quad + r;
              if (fr < nyl) part[o0 + (size_t)fr * P.nx + 16 * nt + c16] = o[r];
            }
          }
        };
        store();
        // A zero weight must not carry an infinity or NaN of a far column or of a row's
        // overflowing sum to a node.  Either is in every output of its columns then, and
        // the plane is summed without the matrix cores, zero weights left out.
        float fin = 0.f;   // stays 0 if every output is finite, else turns NaN
#pragma unroll
        for (int r = 0; r < 4; ++r) fin = fmaf(o[r], 0.f, fin);
        if (__any(fin != 0.f)) {
          o = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma clang loop unroll(disable)
          for (int rt = 0; rt < RT; ++rt) {
            f32x4 x = (f32x4){0.f, 0.f, 0.f, 0.f};   // sums over x, as acc
#pragma clang loop unroll(disable)
            for (int l = 0; l < BX; ++l) {
              const float w = sWx[nt][l >> 2][16 * (l & 3) + c16];
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float v = V[min(rt * 16 + 4 * quad + r, BY - 1) * VP + l];
                x[r] = w != 0.f ? fmaf(w, v, x[r]) : x[r];
              }
            }
#pragma clang loop unroll(disable)
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float v = __shfl(x[r], 16 * q + c16, 64);   // row 16 rt + 4 q + r
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                  const float w = sWy[mt][4 * rt + r][16 * q + 4 * quad + k];
                  o[k] = w != 0.f ? fmaf(w, v, o[k]) : o[k];
                }
              }
          }
          store();
        }
      }
    }
  };
  // Writes one node plane (local index kloc) of the transposed conversion: the
  // per-column sums go to LDS and, behind one barrier, one wave per component and 16
  // node columns reduces them; the others go on.  sV is written again only behind a
  // later barrier.
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), tasks = 3 * ((nxl + 15) / 16);
  auto flush = [&](const float (&acc)[3], int kloc) {
    if constexpr (NEED_C) {   // (only the derivative modes gather)
#pragma unroll
      for (int d = 0; d < 3; ++d) sV[d][ty * VP + tx] = inC ? acc[d] : 0.f;
      __syncthreads();
      for (int w = wave; w < tasks; w += NT / 64) reduce(kloc, w % 3, w / 3);
      if constexpr (SSD) __syncthreads();
    }
  };

  // Register windows of the own column; slot (t - tfirst) mod 3.
  float Tw[3] = {0.f, 0.f, 0.f}, Rv[3] = {0.f, 0.f, 0.f}, av[3] = {0.f, 0.f, 0.f};
  float dzT[3] = {0.f, 0.f, 0.f}, dzR[3] = {0.f, 0.f, 0.f};   // differences to the plane before
  float g[3][3] = {{0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}, {0.f, 0.f, 0.f}};
  float e0[3] = {0.f, 0.f, 0.f}, ezp[3] = {0.f, 0.f, 0.f};
  float acc_lo[3] = {0.f, 0.f, 0.f}, acc_hi[3] = {0.f, 0.f, 0.f};
  int KL = noz;
  double obj = 0.0;

  // xy-interpolated u and p at the two node planes bracketing the current plane,
  // and their differences (the z interpolation of every plane in between is one FMA)
  int Kp = -0x7fffffff;
  float ulo[3] = {0.f, 0.f, 0.f}, udz[3] = {0.f, 0.f, 0.f};
  float plo[3] = {0.f, 0.f, 0.f}, pdz[3] = {0.f, 0.f, 0.f};
  // template and reference through buffer descriptors: the corner loads share one
  // vector offset, the reference load needs only the plane's scalar offset
  const __amdgpu_buffer_rsrc_t rsT = raw_buffer(P.Tp, P.Tbytes), rsR = raw_buffer(P.R, P.Rbytes);
  const CornerOffsets co{4u * (unsigned)P.PX, 4u * (unsigned)P.PXY, 4u * (unsigned)(P.PX + P.PXY)};
  const unsigned rcol = colxy << 2;
  auto xy_interp = [&](const float* __restrict__ f, int k, const Conv1 cvx, const Conv1 cvy, float (&o)[3]) {
    const float wx0 = 1.0f - cvx.f, wx1 = cvx.f, wy0 = 1.0f - cvy.f, wy1 = cvy.f;
    const unsigned i00 = (unsigned)k * nxy + (unsigned)(cvy.n0 * P.nx + cvx.n0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const unsigned b = (unsigned)d * nb + i00;
      const float lo = fmaf(wx1, ld32(f, b + 1), wx0 * ld32(f, b));
      const float hi = fmaf(wx1, ld32(f, b + nxu + 1), wx0 * ld32(f, b + nxu));
      o[d] = fmaf(wy1, hi, wy0 * lo);
    }
  };
  // The next node plane through LDS: loaded when the march enters a cell, written to
  // LDS in the step behind (the loads precede that step's template loads, which it
  // waits for anyway), read when it enters the next cell.  Cells of two planes or more
  // (P.zcells2), so a barrier lies between each two of these; the loads' latency, which
  // every wave of the group would meet at the same step, is hidden.
  const int nn = nxl * nyl;
  // (a march of fewer than four cells has too little of it to hide for the set-up)
  const bool staged =
      Sm::STG && P.zcells2 && 3 * nn <= 2 * NT && P.cz[min(ze + 1, P.mz - 1)].n0 - P.cz[max(zb - 2, 0)].n0 >= 4;
  float stu[2] = {0.f, 0.f}, stp[2] = {0.f, 0.f};
  bool pending = false;
  auto stage_load = [&](int k) {
    if (k >= P.nz) return;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (tid + i * NT < 3 * nn) {
        const unsigned q = S.sSrc[i][tid] + (unsigned)k * nxy;
        stu[i] = ld32(u, q);
        if (HV) stp[i] = ld32(pv, q);
      }
    pending = true;
  };
  auto stage_store = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
      if (tid + i * NT < 3 * nn) {
        S.sN[0][tid + i * NT] = stu[i];
        if (HV) S.sN[HV ? 1 : 0][tid + i * NT] = stp[i];
      }
    pending = false;
  };
  auto staged_interp = [&](const float* f, const Conv1 cvx, const Conv1 cvy, float (&o)[3]) {
    const float wx0 = 1.0f - cvx.f, wx1 = cvx.f, wy0 = 1.0f - cvy.f, wy1 = cvy.f;
    const float* q = f + (cvy.n0 - noy) * nxl + (cvx.n0 - nox);
#pragma unroll
    for (int d = 0; d < 3; ++d, q += nn) {
      const float lo = fmaf(wx1, q[1], wx0 * q[0]);
      const float hi = fmaf(wx1, q[nxl + 1], wx0 * q[nxl]);
      o[d] = fmaf(wy1, hi, wy0 * lo);
    }
  };
  if constexpr (Sm::STG)
    if (staged) {
      for (int i = 0; i < 2; ++i) {
        const int e = tid + i * NT, d = e / nn, r = e - d * nn, row = r / nxl;
        S.sSrc[i][tid] = (unsigned)d * nb + (unsigned)((noy + row) * P.nx + nox + r - row * nxl);
      }
      stage_load(P.cz[max(zb - 2, 0)].n0 + 2);
      if (pending) stage_store();
      __syncthreads();
    }

  // Stage A inputs of the next plane, loaded one step ahead.
  float nx_t[8];
  float nx_fx = 0.f, nx_fy = 0.f, nx_fz = 0.f, nx_R = 0.f;
  float nx_pp[3] = {0.f, 0.f, 0.f};
  auto issue = [&](int tt) {
    const int tc = min(max(tt, 0), P.mz - 1);
    const int jz = tt - zb + 2;   // LDS slot of plane tt (entries are clamped into the image)
    Conv1 cvz = sCz[jz];
    cvz.n0 = __builtin_amdgcn_readfirstlane(cvz.n0);   // uniform: keeps the plane logic scalar
    cvz.f = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, cvz.f)));
    if (cvz.n0 != Kp) {
      int ct = tid;   // (opaque, so that nothing of the column's weights is kept over the march)
      asm volatile("" : "+v"(ct));
      const Conv1 cvx = sCx[ct % BX], cvy = sCy[ct / BX];
      float uhi[3], phi[3];
      bool next = cvz.n0 == Kp + 1;
      if (next) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          ulo[d] = S.sHi[d][ct];
          if (HV) plo[d] = S.sHi[HV ? 3 + d : 0][ct];
        }
      } else {
        xy_interp(u, cvz.n0, cvx, cvy, ulo);
        if (HV) xy_interp(pv, cvz.n0, cvx, cvy, plo);
      }
      if (Sm::STG && staged && next) {
        staged_interp(S.sN[0], cvx, cvy, uhi);
        if (HV) staged_interp(S.sN[HV ? 1 : 0], cvx, cvy, phi);
        stage_load(cvz.n0 + 2);
      } else {
        xy_interp(u, cvz.n0 + 1, cvx, cvy, uhi);
        if (HV) xy_interp(pv, cvz.n0 + 1, cvx, cvy, phi);
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        S.sHi[d][ct] = uhi[d];
        udz[d] = uhi[d] - ulo[d];
        if (HV) {
          S.sHi[HV ? 3 + d : 0][ct] = phi[d];
          pdz[d] = phi[d] - plo[d];
        }
      }
      Kp = cvz.n0;
    }
    const float fz = cvz.f;
    const float qx = template_pos(spx.frac, fmaf(fz, udz[0], ulo[0]), P.ihTx, nx_fx);
    const float qy = template_pos(spy.frac, fmaf(fz, udz[1], ulo[1]), P.ihTy, nx_fy);
    const Samp1 spz = sSz[jz];
    const float qz = template_pos(spz.frac, fmaf(fz, udz[2], ulo[2]), P.ihTz, nx_fz);
    const unsigned kx = (unsigned)clamp_lo0(bx2 + floor_to_int(qx), P.mTx + 2);
    const unsigned ky = (unsigned)clamp_lo0(by2 + floor_to_int(qy), P.mTy + 2);
    const unsigned kz = (unsigned)clamp_lo0(spz.base + floor_to_int(qz), P.mTz + 2);
    unsigned v;
    if (mul24)
      v = __umul24(kz, pxy4) + __umul24(ky, px4);
    else {
      asm volatile("");   // (a branch: the full multiplies stay out of the common path)
      v = kz * pxy4 + ky * px4;
    }
    v += kx << 2;
    {
      const FPair a = buf_ld2(rsT, v, 0), b = buf_ld2(rsT, v, co.row), c = buf_ld2(rsT, v, co.plane),
                  d = buf_ld2(rsT, v, co.both);
      nx_t[0] = a.a;
      nx_t[1] = a.b;
      nx_t[2] = b.a;
      nx_t[3] = b.b;
      nx_t[4] = c.a;
      nx_t[5] = c.b;
      nx_t[6] = d.a;
      nx_t[7] = d.b;
    }
    nx_R = buf_ld(rsR, rcol, (unsigned)tc * plane * 4u);
    if (HV) {
#pragma unroll
      for (int d = 0; d < 3; ++d) nx_pp[d] = fmaf(fz, pdz[d], plo[d]);
    }
  };

  // Rows are formed at planes zb - 1 .. ze, of which the image's first chunk has no
  // plane -1: two steps of stage A alone, then all three stages per step.
  const int tfirst = max(zb - 2, -1), tlast = ze + 1;

  auto step = [&](auto Kc, auto Lead, int t) {
    constexpr int K = decltype(Kc)::value;   // slot of plane t
    constexpr int K1 = (K + 2) % 3;          // slot of plane t-1
    constexpr int K2 = (K + 1) % 3;          // slot of plane t-2

    if (Sm::STG && pending) stage_store();

    // ---------------- stage A: plane t ----------------
    {
      const Tri s = trilinear(P, nx_t, nx_fx, nx_fy, nx_fz);
      Tw[K] = s.v;
      g[K][0] = s.gx;
      g[K][1] = s.gy;
      g[K][2] = s.gz;
      Rv[K] = nx_R;
      dzT[K] = Tw[K] - Tw[K1];
      dzR[K] = Rv[K] - Rv[K1];
      if (HV) av[K] = fmaf(s.gx, nx_pp[0], fmaf(s.gy, nx_pp[1], s.gz * nx_pp[2]));
      if constexpr (!SSD) {
        const int sl = t & 1;
        sTw[sl][XP + tid] = Tw[K];
        sR[sl][XP + tid] = Rv[K];
        if (HV) sA[sl][XP + tid] = av[K];
      }
    }
    if (t < tlast) issue(t + 1);
    // No barrier here: stage B reads only LDS slots of plane t-1 (written in the
    // previous step) and the slots written above were last read before the
    // barrier that ends the previous step.

    if constexpr (decltype(Lead)::value) {
      if constexpr (!SSD) __syncthreads();
      return;
    }

    // ---------------- stage B: plane zc = t-1 ----------------
    const int zc = t - 1;
    float ezm = 0.f;
    if constexpr (SSD) {
      const float r = Tw[K1] - Rv[K1];
      if (MODE != MODE_HV && inB && zc >= zb && zc < ze) {
        const double rd = r;
        obj += 0.5 * rd * rd;
      }
      if constexpr (NEED_C) e0[K1] = inB ? (HV ? av[K1] : r) : 0.f;
    } else {
      // Every lane evaluates the row (ring columns and columns outside the image
      // read finite neighbours: clamped samples or the zero pads), and a lane
      // that does not own its row scales the products by 0: no divergent branch
      // and no per-step clearing of the products.  The row plane behind the image's
      // last one gets 1 / |grad T|^2 = 0 instead, which zeroes its products.
      const int s1 = zc & 1;
      const int q = XP + tid;
      const float Tc = Tw[K1], Rc = Rv[K1];
      const float dTxm = sTw[s1][q - 1] - Tc, dTxp = sTw[s1][q + 1] - Tc;
      const float dTym = sTw[s1][q - BX] - Tc, dTyp = sTw[s1][q + BX] - Tc;
      const float dTzm = -dzT[K1], dTzp = dzT[K];
      const float dRxm = sR[s1][q - 1] - Rc, dRxp = sR[s1][q + 1] - Rc;
      const float dRym = sR[s1][q - BX] - Rc, dRyp = sR[s1][q + BX] - Rc;
      const float dRzm = -dzR[K1], dRzp = dzR[K];
      const float tau2 = zc < P.mz ? P.tau2 : __builtin_inff();
      const float nT2 = fmaf(fmaf(dTxm, dTxm, dTxp * dTxp), P.hhx,
                             fmaf(fmaf(dTym, dTym, dTyp * dTyp), P.hhy,
                                  fmaf(fmaf(dTzm, dTzm, dTzp * dTzp), P.hhz, tau2)));
      const float nR2 = fmaf(fmaf(dRxm, dRxm, dRxp * dRxp), P.hhx,
                             fmaf(fmaf(dRym, dRym, dRyp * dRyp), P.hhy,
                                  fmaf(fmaf(dRzm, dRzm, dRzp * dRzp), P.hhz, P.rho2)));
      const float r1 = fmaf(fmaf(dTxm, dRxm, dTxp * dRxp), P.hhx,
                            fmaf(fmaf(dTym, dRym, dTyp * dRyp), P.hhy,
                                 fmaf(fmaf(dTzm, dRzm, dTzp * dRzp), P.hhz, P.taurho)));
      // 1 - r^2 from the float32 sums in float64: in float32 it cancels where r is
      // close to 1 (aligned images), and the bias of the hardware reciprocal would
      // add up over the voxels of the objective sum
      if (MODE != MODE_HV && inB && zc >= zb && zc < ze)
        obj += 1.0 - ((double)r1 * (double)r1) / ((double)nT2 * (double)nR2);
      if constexpr (NEED_C) {
        // rows rho-hat(k) = q(k) / (|grad T| |grad R|): every product that leaves the
        // stage holds two of them, so no square root is formed (the host scales the
        // squared norms, r1 and q by about 1 / (tau rho), which cancels)
        const float rT = rcp_norm(nT2), rR = rcp_norm(nR2);
        const float c2 = r1 * rT;
        const float qxm = P.hhx * fmaf(-c2, dTxm, dRxm), qxp = P.hhx * fmaf(-c2, dTxp, dRxp);
        const float qym = P.hhy * fmaf(-c2, dTym, dRym), qyp = P.hhy * fmaf(-c2, dTyp, dRyp);
        const float qzm = P.hhz * fmaf(-c2, dTzm, dRzm), qzp = P.hhz * fmaf(-c2, dTzp, dRzp);
        const float q0 = -(((qxm + qxp) + (qym + qyp)) + (qzm + qzp));
        float z;   // z_l times |grad T| |grad R|
        if constexpr (HV) {
          z = q0 * av[K1];
          z = fmaf(qxm, sA[s1][q - 1], z);
          z = fmaf(qxp, sA[s1][q + 1], z);
          z = fmaf(qym, sA[s1][q - BX], z);
          z = fmaf(qyp, sA[s1][q + BX], z);
          z = fmaf(qzm, av[K2], z);
          z = fmaf(qzp, av[K], z);
        } else {
          z = r1;
        }
        const float w = own_row * (rR * (rT * z));   // (this order: the factors alone may overflow)
        sE[s1][0][EP + tid] = qxp * w;
        sE[s1][1][EP + tid] = qxm * w;
        sE[s1][2][EP + tid] = qyp * w;
        sE[s1][3][EP + tid] = qym * w;
        ezp[K1] = qzp * w;
        ezm = qzm * w;
        e0[K1] = q0 * w;
      }
    }

    // ---------------- stage C: plane c = t-2 ----------------
    if constexpr (NEED_C) {
      const int c = t - 2;
      if (c >= zb && c < ze) {
        Conv1 cvz = sCz[c - zb + 2];
        cvz.n0 = __builtin_amdgcn_readfirstlane(cvz.n0);
        cvz.f = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, cvz.f)));
        if (cvz.n0 != KL) {  // node plane KL is complete
          flush(acc_lo, KL - noz);
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            acc_lo[d] = acc_hi[d];
            acc_hi[d] = 0.f;
          }
          KL = cvz.n0;
        }
        {
          float w = e0[K2];
          if constexpr (!SSD) {
            // rows of the neighbours within the group (beyond its edge: the zero pad,
            // or a ring column of the next row, which holds 0)
            const int s2 = c & 1;
            w += sE[s2][1][EP + tid + 1];
            w += sE[s2][0][EP + tid - 1];
            w += sE[s2][3][EP + tid + BX];
            w += sE[s2][2][EP + tid - BX];
            w += ezm;
            w += ezp[K];
          }
          const float w1 = cvz.f * w, w0 = (1.0f - cvz.f) * w;
#pragma unroll
          for (int d = 0; d < 3; ++d) {
            acc_lo[d] = fmaf(w0, g[K2][d], acc_lo[d]);
            acc_hi[d] = fmaf(w1, g[K2][d], acc_hi[d]);
          }
        }
      }
    }
    // SSD exchanges nothing between columns within a step (flush has its own barriers)
    if constexpr (!SSD) __syncthreads();
  };

  using std::integral_constant;
  issue(tfirst);
  step(integral_constant<int, 0>{}, std::true_type{}, tfirst);
  step(integral_constant<int, 1>{}, std::true_type{}, tfirst + 1);
  for (int t = tfirst + 2; t <= tlast; t += 3) {
    step(integral_constant<int, 2>{}, std::false_type{}, t);
    if (t + 1 <= tlast) step(integral_constant<int, 0>{}, std::false_type{}, t + 1);
    if (t + 2 <= tlast) step(integral_constant<int, 1>{}, std::false_type{}, t + 2);
  }

  if constexpr (NEED_C) {
    flush(acc_lo, KL - noz);
    __syncthreads();
    flush(acc_hi, KL + 1 - noz);
  }
  if constexpr (MODE != MODE_HV) block_sum_store<NT>(obj, P.red + bid, sRed);
}

// Bound by vector-instruction issue (about 190 per step and wave, 0.87 of the cycles at
// 512x512x900 voxels), so the steps hold no instruction that a table, a uniform branch
// or the order of the factors can save: rows without their common factor 1 / (|grad T|
// |grad R|), which enters squared and needs no square root; z differences formed
// once; two lead steps of stage A alone instead of zeroed products.  205 -> 190
// instructions, Hessian product 512x512x900 1951 -> 1879 us, ten pairs of up to
// 512x512x136 1866 -> 1825 us; 128 registers (two groups per CU) hold because what is
// read once per cell lies in LDS.
// Node values through LDS a node plane ahead: 24 loads per cell, column and wave, whose
// latency all waves of a group met at the same step, become one or two per thread:
// 1879 -> 1800 us, ten pairs 1825 -> 1765 us (8-byte loads of node pairs instead: 2075
// us; the template's corner pairs as 4-byte loads: 1947 us).
template <int BX, int BY, int MODE, bool SSD>
__global__ __launch_bounds__(BX* BY) __attribute__((amdgpu_waves_per_eu(4))) void ngf_tile_kernel(
    const TileParams P, const float* __restrict__ u, const float* __restrict__ pv) {
  if (P.live && !ld_coherent(P.live)) return;   // a device-steered solve has stopped
  __shared__ TileSmem<BX, BY, MODE, SSD> S;
  tile_body<BX, BY, MODE, SSD>(P, xcd_block_id(), u, pv, S);
}

// The tiles of a batch of problems in one launch, a group per tile.  A tile's results
// depend only on its problem and tile id, so the output equals one launch per
// problem bit for bit.  At most 128 VGPRs (four waves per SIMD): two groups of 512
// threads per CU, as for the single-problem kernel.  The hardware hands out the
// groups as they end, so a work counter of resident groups adds nothing but its
// clearing, an atomic, two barriers per tile and the registers of its loop (ten pairs
// of up to 512x512x136 voxels 1869 us with it, 1866 us without).
template <int BX, int BY, int MODE>
__global__ __launch_bounds__(BX* BY) __attribute__((amdgpu_waves_per_eu(4))) void ngf_tile_batch_kernel(const BatchJobs J) {
  __shared__ TileSmem<BX, BY, MODE, false> S;
  const int item = blockIdx.x;
  int pr = 0;
  while (pr + 1 < J.n && J.prefix[pr + 1] <= item) ++pr;
  if (J.active && !ld_coherent(J.active + pr)) return;
  const BatchJob& jb = J.jobs[pr];
  const int first = J.prefix[pr];   // every XCD takes a part of every problem
  tile_body<BX, BY, MODE, false>(jb.t, xcd_remap(item - first, J.prefix[pr + 1] - first), jb.u, jb.p, S);
}

template <int BX, int BY, bool SSD>
static void launch_tile_dist(int mode, const TileParams& p, const float* u, const float* pv, int grid,
                             hipStream_t st) {
  dim3 blk(BX * BY), grd(grid);
  switch (mode) {
    case MODE_OBJ:
      hipLaunchKernelGGL((ngf_tile_kernel<BX, BY, MODE_OBJ, SSD>), grd, blk, 0, st, p, u, pv);
      break;
    case MODE_GRAD:
      hipLaunchKernelGGL((ngf_tile_kernel<BX, BY, MODE_GRAD, SSD>), grd, blk, 0, st, p, u, pv);
      break;
    default:
      hipLaunchKernelGGL((ngf_tile_kernel<BX, BY, MODE_HV, SSD>), grd, blk, 0, st, p, u, pv);
      break;
  }
}

template <int BX, int BY>
static hipError_t launch_tile_shape(int mode, const TileParams& p, const float* u, const float* pv,
                                    int grid, hipStream_t st) {
  if (p.ssd)
    launch_tile_dist<BX, BY, true>(mode, p, u, pv, grid, st);
  else
    launch_tile_dist<BX, BY, false>(mode, p, u, pv, grid, st);
  return hipGetLastError();
}

template <int BX, int BY>
static hipError_t launch_tile_batch_shape(int mode, const BatchJobs& j, hipStream_t st) {
  if (j.total <= 0) return hipSuccess;
  dim3 blk(BX * BY), grd(j.total);
  switch (mode) {
    case MODE_OBJ:
      hipLaunchKernelGGL((ngf_tile_batch_kernel<BX, BY, MODE_OBJ>), grd, blk, 0, st, j);
      break;
    case MODE_GRAD:
      hipLaunchKernelGGL((ngf_tile_batch_kernel<BX, BY, MODE_GRAD>), grd, blk, 0, st, j);
      break;
    default:
      hipLaunchKernelGGL((ngf_tile_batch_kernel<BX, BY, MODE_HV>), grd, blk, 0, st, j);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_tile(const TileShape& s, int mode, const TileParams& p, const float* u,
                       const float* pv, int grid, hipStream_t st) {
  if (s.bx == 32 && s.by == 16) return launch_tile_shape<32, 16>(mode, p, u, pv, grid, st);
  if (s.bx == 64 && s.by == 8) return launch_tile_shape<64, 8>(mode, p, u, pv, grid, st);
  if (s.bx == 32 && s.by == 32) return launch_tile_shape<32, 32>(mode, p, u, pv, grid, st);
  if (s.bx == 64 && s.by == 16) return launch_tile_shape<64, 16>(mode, p, u, pv, grid, st);
  return hipErrorInvalidValue;
}

hipError_t launch_tile_batch(const TileShape& s, int mode, const BatchJobs& j, hipStream_t st) {
  if (s.bx == 32 && s.by == 16) return launch_tile_batch_shape<32, 16>(mode, j, st);
  if (s.bx == 64 && s.by == 8) return launch_tile_batch_shape<64, 8>(mode, j, st);
  if (s.bx == 32 && s.by == 32) return launch_tile_batch_shape<32, 32>(mode, j, st);
  if (s.bx == 64 && s.by == 16) return launch_tile_batch_shape<64, 16>(mode, j, st);
  return hipErrorInvalidValue;
}

}  // namespace mfr
