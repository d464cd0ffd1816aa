// Grid gradient dL/dF and the transform gradient through the trilinear
// weights (the adjoint of Eq. (2)), gathered per cell instead of scattered
// per point.  k_block_pull (the default): one wave owns a block of cells of one
// grid, maps the block's box back to global space (inverse of the transform of
// Eq. (1)), walks the points of the spatial bins that overlap it, keeps those
// whose float32 cell decision lies in the block, and forms the block's vertex
// sums of w_q * dL/dy_c with matrix instructions.  k_cell_pull: one thread owns
// one cell and sums its 8 corners in registers.  A second kernel adds, for each
// vertex, the sums of its (up to 8) blocks or cells.  No atomics; every sum has
// a fixed order.

namespace apmg {

struct CellArgs {
  Shape s;
  const float* G; size_t G_stride;      // [M][12] per model
  const void* F; size_t F_stride;       // grids (corner values for the transform gradient)
  const float4* pts4; int64_t n;        // sorted points [model][n] as (x, y, z, 0)
  const uint32_t* start;                // [model][NB^3 + 1]
  const float* dY;                      // [model][grid][n][C] at model * dY_stride + grid * dY_grid
  size_t dY_stride, dY_grid;
  float* CC;                            // k_cell_pull: [model][M][8][(R-1)^3][C] (corner-major);
                                        // k_block_pull: the blocks' vertex lattices
  double* dGpart;                       // [model][M][nblk][12] (DG)
  const int32_t* active;
  int nblk;                             // blocks of 256 cells per grid; launch nmodels * M * nblk blocks
  double cell;                          // 2 / (R - 1): the width of a cell in local coordinates
  int Rt;                               // 4-D grids (two time slices per cell): time vertices
};

// Corner weight q = a + 2b + 4c of the trilinear weights of offsets w.  The per-cell gather adds
// round(w_q * dL/dy) to the corner sums (a product, then a sum: no fused multiply-add).
__device__ inline float corner_weight(int qq, const float w[3]) {
  return ((qq & 1) ? w[0] : 1.f - w[0]) * ((qq & 2) ? w[1] : 1.f - w[1]) * ((qq & 4) ? w[2] : 1.f - w[2]);
}
__device__ inline float corner_product(float wq, float d) {
#pragma clang fp contract(off)
  return wq * d;
}
__device__ inline float add_rounded(float acc, float v) {
#pragma clang fp contract(off)
  return acc + v;
}

// 1 / x in float64 for a normal x: the hardware estimate and two Newton steps.
__device__ inline double recip_f64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
  return __builtin_fma(__builtin_fma(-x, r, 1.0), r, r);
}

// The local box of the cells [c0, c0 + w) (w cells per axis, clipped to the grid) minus the
// translation, widened by 1e-4 (covers the float32 rounding of the cell decision), in float64.
// cell = 2 / R1, the width of a cell.
__device__ inline void local_box(const float* Gg, const int c0[3], const int w[3], int R1, double cell, double blo[3],
                                 double bhi[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const int e = min(c0[d] + w[d], R1);
    blo[d] = -1.0 + cell * c0[d] - 1e-4 - (double)Gg[4 * d + 3];
    bhi[d] = -1.0 + cell * e + 1e-4 - (double)Gg[4 * d + 3];
  }
}

// Tighter x-range [x0, x1] (bins, within [lo0, hi0]) of the bin row (yb, zb) for a local box:
// the x for which some (y, z) of the row satisfies each of the three slab constraints
// blo_d <= A_d . x <= bhi_d, taken one slab at a time (a superset of the exact range), in
// float64, with the row widened by 1e-5 (the float32 rounding of the binning) and the x-range
// by 1e-4.  The edge rows of the bin grid reach to infinity, because the binning clamps points
// outside the domain into them.  Returns false for an empty row.
// ra[d] = 1 / Gg[4 d] (0 where that coefficient is 0), from span_recips once per transform:
// the x-range's bounds are multiplied by it rather than divided (they are padded anyway).
__device__ inline void span_recips(const float* Gg, double ra[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) ra[d] = Gg[4 * d] != 0.f ? recip_f64((double)Gg[4 * d]) : 0.0;
}
__device__ inline bool row_x_span(const float* Gg, const double ra[3], const double blo[3], const double bhi[3],
                                  int lo0, int hi0, int yb, int zb, int& x0, int& x1) {
  constexpr double kInf = __builtin_inf(), kW = 2.0 / kBinsPerAxis;
  const double ylo = yb == 0 ? -kInf : -1.0 + yb * kW - 1e-5;
  const double yhi = yb == kBinsPerAxis - 1 ? kInf : -1.0 + (yb + 1) * kW + 1e-5;
  const double zlo = zb == 0 ? -kInf : -1.0 + zb * kW - 1e-5;
  const double zhi = zb == kBinsPerAxis - 1 ? kInf : -1.0 + (zb + 1) * kW + 1e-5;
  double xl = -kInf, xh = kInf;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double a0 = Gg[4 * d], a1 = Gg[4 * d + 1], a2 = Gg[4 * d + 2];
    // range of a1 y + a2 z over the row (a zero coefficient contributes exactly 0)
    const double m_lo = (a1 > 0 ? a1 * ylo : a1 < 0 ? a1 * yhi : 0.0) + (a2 > 0 ? a2 * zlo : a2 < 0 ? a2 * zhi : 0.0);
    const double m_hi = (a1 > 0 ? a1 * yhi : a1 < 0 ? a1 * ylo : 0.0) + (a2 > 0 ? a2 * zhi : a2 < 0 ? a2 * zlo : 0.0);
    const double P = blo[d] - m_hi, Q = bhi[d] - m_lo;      // P <= a0 x <= Q
    if (a0 > 0) { xl = fmax(xl, P * ra[d]); xh = fmin(xh, Q * ra[d]); }
    else if (a0 < 0) { xl = fmax(xl, Q * ra[d]); xh = fmin(xh, P * ra[d]); }
    else if (P > 0.0 || Q < 0.0) return false;
  }
  if (!(xl <= xh)) return false;
  const double f0 = floor((xl - 1e-4 + 1.0) * (0.5 * kBinsPerAxis));
  const double f1 = floor((xh + 1e-4 + 1.0) * (0.5 * kBinsPerAxis));
  x0 = (int)fmin(fmax(f0, (double)lo0), (double)hi0);
  x1 = (int)fmin(fmax(f1, (double)lo0), (double)hi0);
  return true;
}

// The adjoint of Eq. (2) with respect to the local coordinates for one point of a cell with
// corner values val and offsets w: dl_d = sum_c dL/dy_c d(trilerp_c)/du_d, then the transform
// gradient terms (dl h) x^T and (dl h) added to gacc (x masked to 0 for a rejected candidate,
// which may be a NaN point and has dL/dy = 0).
template <int C>
__device__ inline void add_transform_grad(const float val[8][C], const float wu[3], const float dyv[C], float hR,
                                          bool ok, float px, float py, float pz, float gacc[12]) {
  float dl[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const float ax00 = val[1][c] - val[0][c], ax10 = val[3][c] - val[2][c];
    const float ax01 = val[5][c] - val[4][c], ax11 = val[7][c] - val[6][c];
    const float gx = (1.f - wu[2]) * ((1.f - wu[1]) * ax00 + wu[1] * ax10) +
                     wu[2] * ((1.f - wu[1]) * ax01 + wu[1] * ax11);
    const float x00 = __builtin_fmaf(wu[0], ax00, val[0][c]);
    const float x10 = __builtin_fmaf(wu[0], ax10, val[2][c]);
    const float x01 = __builtin_fmaf(wu[0], ax01, val[4][c]);
    const float x11 = __builtin_fmaf(wu[0], ax11, val[6][c]);
    const float gy = (1.f - wu[2]) * (x10 - x00) + wu[2] * (x11 - x01);
    const float y0 = __builtin_fmaf(wu[1], x10 - x00, x00);
    const float y1 = __builtin_fmaf(wu[1], x11 - x01, x01);
    dl[0] = __builtin_fmaf(dyv[c], gx, dl[0]);
    dl[1] = __builtin_fmaf(dyv[c], gy, dl[1]);
    dl[2] = __builtin_fmaf(dyv[c], y1 - y0, dl[2]);
  }
  const float xs[4] = {ok ? px : 0.f, ok ? py : 0.f, ok ? pz : 0.f, 1.f};
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int k = 0; k < 4; ++k) gacc[4 * r + k] = __builtin_fmaf(dl[r] * hR, xs[k], gacc[4 * r + k]);
}

// Block order: xcd_logical over (model, cell block, grid), so an XCD works through a slab of
// cells for all grids at once and the points of that slab stay in its L2.

// Candidates are taken U at a time (U = 2, 4 or 8, a launch-shape choice): their
// coordinates (and, for the accepted ones, dL/dy) are loaded together, and a rejected
// candidate adds exact zeros, so the sums keep the candidate order with no branch per point.
template <int C, bool GF16, bool DG, int U>
__global__ void __launch_bounds__(256) k_cell_pull(CellArgs a) {
  constexpr int kCellUnroll = U;
  __shared__ float sG[12];
  __shared__ float sInv[9];
  __shared__ int sBad;
  __shared__ double sred[4][12];
  const Shape s = a.s;
  const int64_t per_model = (int64_t)a.nblk * s.M;
  const int64_t L = xcd_logical(blockIdx.x, gridDim.x);
  const int model = (int)(L / per_model);
  const int blk = (int)((L % per_model) / s.M), g = (int)(L % s.M);
  const bool act = !a.active || a.active[model];
  const int R1 = s.R - 1;
  const int64_t ncell = (int64_t)R1 * R1 * R1;
  if (threadIdx.x < 12) sG[threadIdx.x] = a.G[model * a.G_stride + 12 * g + threadIdx.x];
  __syncthreads();
  if (threadIdx.x == 0) {
    // inverse of the 3x3 block, float64
    double A[3][3];
    for (int r = 0; r < 3; ++r) for (int c = 0; c < 3; ++c) A[r][c] = sG[4 * r + c];
    const double c00 = A[1][1] * A[2][2] - A[1][2] * A[2][1], c01 = A[1][2] * A[2][0] - A[1][0] * A[2][2];
    const double c02 = A[1][0] * A[2][1] - A[1][1] * A[2][0];
    const double det = A[0][0] * c00 + A[0][1] * c01 + A[0][2] * c02;
    const double inv[9] = {c00, A[0][2] * A[2][1] - A[0][1] * A[2][2], A[0][1] * A[1][2] - A[0][2] * A[1][1],
                           c01, A[0][0] * A[2][2] - A[0][2] * A[2][0], A[0][2] * A[1][0] - A[0][0] * A[1][2],
                           c02, A[0][1] * A[2][0] - A[0][0] * A[2][1], A[0][0] * A[1][1] - A[0][1] * A[1][0]};
    int bad = !(fabs(det) > 1e-30);
    for (int k = 0; k < 9; ++k) {
      const double v = inv[k] / det;
      sInv[k] = (float)v;
      bad |= !isfinite((float)v);
    }
    sBad = bad;
  }
  __syncthreads();
  const int64_t cell = (int64_t)blk * blockDim.x + threadIdx.x;
  const bool valid = act && cell < ncell;
  float acc[8][C];
#pragma unroll
  for (int q = 0; q < 8; ++q)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[q][c] = 0.f;
  float gacc[DG ? 12 : 1];
#pragma unroll
  for (int k = 0; k < (DG ? 12 : 1); ++k) gacc[k] = 0.f;
  const float4* P4 = a.pts4 + (size_t)model * a.n;
  const float* dY = a.dY + model * a.dY_stride + g * a.dY_grid;
  const uint32_t* start = a.start + (size_t)model * (kBinsPerAxis * kBinsPerAxis * kBinsPerAxis + 1);
  if (valid) {
    const int cx = (int)(cell % R1), cy = (int)((cell / R1) % R1), cz = (int)(cell / ((int64_t)R1 * R1));
    const float hR = 0.5f * (float)R1;
    // bins overlapping the cell's box in global space; the 1e-4 margin (world units) covers the
    // float32 rounding of the cell decision (~1e-6) and of this box
    int lo[3], hi[3];
    if (sBad) {
      for (int d = 0; d < 3; ++d) { lo[d] = 0; hi[d] = kBinsPerAxis - 1; }
    } else {
      const float lm[3] = {-1.f + (2.f * cx + 1.f) / R1 - sG[3], -1.f + (2.f * cy + 1.f) / R1 - sG[7],
                           -1.f + (2.f * cz + 1.f) / R1 - sG[11]};
      const float hl = 1.0f / R1;
      for (int d = 0; d < 3; ++d) {
        const float wc = sInv[3 * d] * lm[0] + sInv[3 * d + 1] * lm[1] + sInv[3 * d + 2] * lm[2];
        const float hw = (fabsf(sInv[3 * d]) + fabsf(sInv[3 * d + 1]) + fabsf(sInv[3 * d + 2])) * hl;
        const float b0 = floorf((wc - hw - 1e-4f + 1.f) * (0.5f * kBinsPerAxis));
        const float b1 = floorf((wc + hw + 1e-4f + 1.f) * (0.5f * kBinsPerAxis));
        lo[d] = (int)fminf(fmaxf(b0, 0.f), (float)(kBinsPerAxis - 1));
        hi[d] = (int)fminf(fmaxf(b1, 0.f), (float)(kBinsPerAxis - 1));
      }
    }
    float val[DG ? 8 : 1][C];
    if constexpr (DG) {
      const int me[3] = {cx, cy, cz};
      gather_cell<C, GF16>(GF16 ? (const void*)((const __half*)a.F + model * a.F_stride)
                                : (const void*)((const float*)a.F + model * a.F_stride),
                           g, s.R, me, val);
    }
    double blo[3], bhi[3], ra[3];
    const int me0[3] = {cx, cy, cz}, one[3] = {1, 1, 1};
    local_box(sG, me0, one, R1, a.cell, blo, bhi);
    span_recips(sG, ra);
    for (int bz = lo[2]; bz <= hi[2]; ++bz)
      for (int by = lo[1]; by <= hi[1]; ++by) {
        int x0 = lo[0], x1 = hi[0];
        if (!sBad && !row_x_span(sG, ra, blo, bhi, lo[0], hi[0], by, bz, x0, x1)) continue;
        const int row = (bz * kBinsPerAxis + by) * kBinsPerAxis;
        const uint32_t p0 = start[row + x0], p1 = start[row + x1 + 1];
        for (uint32_t p = p0; p < p1; p += kCellUnroll) {
          float4 q[kCellUnroll];
#pragma unroll
          for (int u = 0; u < kCellUnroll; ++u) q[u] = P4[min(p + u, p1 - 1)];
          bool ok[kCellUnroll];
          float w[kCellUnroll][3];
#pragma unroll
          for (int u = 0; u < kCellUnroll; ++u) {
            float l[3];
            local_coords(sG, q[u].x, q[u].y, q[u].z, l);
            int i0[3];
            const bool in = cell_of(l, hR, s.R, i0, w[u]);
            ok[u] = (p + u < p1) && in && i0[0] == cx && i0[1] == cy && i0[2] == cz;
#pragma unroll
            for (int d = 0; d < 3; ++d) w[u][d] = ok[u] ? w[u][d] : 0.f;
          }
          float dy[kCellUnroll][C];
#pragma unroll
          for (int u = 0; u < kCellUnroll; ++u)
#pragma unroll
            for (int c = 0; c < C; ++c) dy[u][c] = ok[u] ? dY[(size_t)(p + u) * C + c] : 0.f;
#pragma unroll
          for (int u = 0; u < kCellUnroll; ++u) {
#pragma unroll
            for (int qq = 0; qq < 8; ++qq) {
              const float wq = corner_weight(qq, w[u]);
#pragma unroll
              for (int c = 0; c < C; ++c) acc[qq][c] = add_rounded(acc[qq][c], corner_product(wq, dy[u][c]));
            }
            if constexpr (DG)
              add_transform_grad<C>(val, w[u], dy[u], hR, ok[u], q[u].x, q[u].y, q[u].z, gacc);
          }
        }
      }
    float* out = a.CC + ((size_t)model * s.M + g) * 8 * ncell * C + cell * C;
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int c = 0; c < C; ++c) out[q * ncell * C + c] = acc[q][c];
  }
  if constexpr (DG) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const double t = wave_sum((double)gacc[k]);
      if (lane == 0) sred[wave][k] = t;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
      const double t = sred[0][threadIdx.x] + sred[1][threadIdx.x] + sred[2][threadIdx.x] + sred[3][threadIdx.x];
      a.dGpart[(((size_t)model * s.M + g) * a.nblk + blk) * 12 + threadIdx.x] = t;
    }
  }
}

// The grid gradient by matrix products, one wave per block of cells of one grid.  A point of
// cell (cx, cy, cz) with offsets w adds w_q dL/dy_c at the cell's 8 corners: the product of a
// hat function per axis, H_v(t) = max(0, 1 - |t - v|) at the block's vertices v (zero at every
// vertex the cell does not touch).  Over the block's points the sums factor into one matrix
// product, D[(vz, vy)][(c, vx)] += sum_p (H_vz H_vy)(p) (H_vx dL/dy_c)(p): 4 x 4 vertices in
// (z, y) are the 16 rows, kVX vertices in x times the C channels (times two time slices for
// the 4-D grids) the columns of v_mfma_f32_16x16x4_f32, whose k dimension takes four points.
// No record is routed to the lane that owns its cell, and a wave holds 4 (8) accumulator
// registers per lane instead of 16 (32).
//
// The wave takes the rows of the bins that overlap the block's box (the union of its cells'
// candidates, each point read once) kRowBatch rows at a time and walks their points as one
// flat sequence, 64 consecutive candidates a step.  Each lane tests its candidate's float32
// cell decision against the block; the lanes that match write the nonzero entries of their
// row and column factors (2 x 2 each; the slots are zero otherwise, and are zeroed again
// after use) to LDS at consecutive slots, element-major, so that one 16-byte read per operand
// feeds four matrix instructions.  Every sum has a fixed order (four slots per instruction,
// instructions in order): bitwise reproducible, though not the plain candidate order of
// k_cell_pull.
//
// What bounds it: the sum of three pipes that overlap only in part.  At 2^20 uniform points,
// 32 grids at 32^3 x 2 (48 M candidates, 30 M matches): vector instructions 0.135 ms (about 90
// per 64 candidates), matrix instructions 0.115 ms (8 cycles of a SIMD per match), LDS 0.15 ms;
// 0.27 ms alone with six waves per SIMD (0.40 ms with four).  The gather it replaced routed each
// match's 16 products through LDS to the lane that owned its cell: bound by vector work, about
// 190 instructions per 64 candidates.  Whole calls, before -> now: the adjoint of 64 grids at
// 64^3 x 4 (2^19 points) 4.25 -> 3.20 ms, 80 brick models a step 7.73 -> 7.11 ms, the 4-D
// forward + adjoint 3.60 -> 3.05 ms.
// Measured and not kept: full (unsparse) factor rows written per match (0.43 ms, 1.7x the vector
// instructions), 64 slots per round (four waves per SIMD).
constexpr int kRowBatch = 64;                // bin rows per batch (one per lane)
constexpr uint32_t kWindow = 4096;           // candidates whose row ends are marked at a time
// The block of cells: kNZ = kNY = 3 cells (4 vertices) in z and y, kVX - 1 cells in x (the axis
// along which a bin row is contiguous): 8 vertices, or 16 for one channel, so that the columns
// fill whole 16-column tiles.
constexpr int kPullNY = 3, kPullNZ = 3;
__host__ __device__ constexpr int pull_vx(int C) { return C == 1 ? 16 : 8; }
__host__ __device__ constexpr int pull_lat(int C) { return 16 * pull_vx(C); }   // vertices of a block's lattice
struct PullBlocks {
  int x, y, z;
  __host__ __device__ int64_t total() const { return (int64_t)x * y * z; }
};
__host__ __device__ inline PullBlocks pull_blocks(int R, int C) {
  const int R1 = R - 1, nx = pull_vx(C) - 1;
  PullBlocks b;
  b.x = (R1 + nx - 1) / nx;
  b.y = (R1 + kPullNY - 1) / kPullNY;
  b.z = (R1 + kPullNZ - 1) / kPullNZ;
  return b;
}

__device__ inline void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// Operand slots in LDS, element-major: element e (0..15, a row or column of a tile) of slot s at
// e * kSlotPitch + s.  Four floats of padding per element row put the 16 bytes that 8 lanes read
// (neighbouring elements, one quad of slots) into distinct banks.  32 slots at a time (a step's
// matches beyond them go in a second round): the wave's LDS is what limits the waves per SIMD.
constexpr int kSlots = 32, kSlotPitch = kSlots + 4;
// Lane k's value of a double, in scalar registers.
__device__ inline double lane_f64(double v, int k) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, k);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), k);
  return __builtin_bit_cast(double, lo | hi << 32);
}

// DG: also the transform gradient of L_rec through the trilinear weights: every lane adds
// the terms of the points it matched (in step order) to its own 12 sums, reduced per
// workgroup in a fixed order into dGpart[model][g][group][12].
// TS = 2: the 4-D grids of Sec. 9, one pass per time cell ("model" index = time cell tc over
// one shared point array sorted by (time cell, bin); start = [tc][NB^3] positions in it, the
// records (x, y, z, t), dL/dy [M][n][C]); a point of cell tc adds (1 - wt) w_q dL/dy to the
// block's slice-0 lattice and wt w_q dL/dy to its slice-1 lattice (time weight wt, Eq. (2)
// extended by linear interpolation in time).
// SPLIT: the four waves of a workgroup share one block (wave w takes steps w, w + 4, ... and the
// four lattices are added in wave order); otherwise each wave has a block of its own.
// Output: lattices CC[model][g][block][vz 4][vy 4][vx][channel + C slice].
// Waves per SIMD: six where the accumulators allow it, four with the transform gradient or four values
// a vertex.  With one channel and the transform gradient (SIX) six hold it too, with 8 values in
// scratch: its matrix work per match is that of two channels, so the gather by itself is bound by
// latency (64 grids at 32^3, 2^19 points, BF16, the whole adjoint: 752 us in the gather per cell owner
// that this one replaced, 830 with four waves, 740 with six).  Four where the waves of a block share it
// (5 grids at 8^3, 43,260 points: 169 us, with six 176) and where the weight products of the 128-wide
// MLP run beside it and take the matrix cores (38 grids at 38^3 binary16, 66,236 points: 320 and 350).
template <int C, bool GF16, bool DG, int TS, bool SPLIT, bool SIX = !DG>
__global__ void __launch_bounds__(256, C == 1 ? (SIX ? 6 : 4) : DG || C * TS > 2 ? 4 : 6) k_block_pull(CellArgs a) {
  static_assert(TS == 1 || (TS == 2 && !DG), "the 4-D pass has no transform gradient");
  constexpr int VX = pull_vx(C), CT = C * TS;
  constexpr int NT = VX * CT / 16;           // 16-column tiles; column = vx CT + channel (+ C slice)
  constexpr int LAT = pull_lat(C) * C * TS;  // floats of a block's lattice
  constexpr int nbk[3] = {VX - 1, kPullNY, kPullNZ};
  // operand slots: the 16 row factors, then the column factors, 16 per tile
  __shared__ float sOp[4][(1 + NT) * 16 * kSlotPitch];
  __shared__ uint64_t sEnd[4][kWindow / 64];  // bit f: candidate f of the window ends a row
  __shared__ uint32_t sDelta[4][kRowBatch + 1];   // per non-empty row: sorted position minus flat index
  __shared__ double sDG[DG ? 4 : 1][12];
  const Shape s = a.s;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int R1 = s.R - 1;
  const PullBlocks nb = pull_blocks(s.R, C);
  const uint32_t nblk_grid = (uint32_t)nb.total();               // cell blocks per grid (the launch fits 2^31)
  const uint32_t groups = SPLIT ? nblk_grid : (nblk_grid + 3) / 4;
  const uint32_t L = xcd_logical32(blockIdx.x, gridDim.x);
  const uint32_t mg = L / s.M, g = L - mg * s.M;                  // (model, group) and grid
  const uint32_t model = mg / groups, grp = mg - model * groups;
  const uint32_t cb = SPLIT ? grp : grp * 4 + __builtin_amdgcn_readfirstlane(wave);   // this wave's cell block
  const bool act = (TS == 2 || !a.active || a.active[model]) && cb < nblk_grid;
  float Gg[12];                                                  // uniform: scalar loads
#pragma unroll
  for (int k = 0; k < 12; ++k) Gg[k] = a.G[model * a.G_stride + 12 * g + k];
  for (int i = 4 * lane; i < (1 + NT) * 16 * kSlotPitch; i += 256) *(f32x4*)(sOp[wave] + i) = f32x4{0.f, 0.f, 0.f, 0.f};
  wave_lds_order();
  f32x4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float gacc[DG ? 12 : 1];
#pragma unroll
  for (int k = 0; k < (DG ? 12 : 1); ++k) gacc[k] = 0.f;
  if (act) {
    // the block's box in global space (inverse of Eq. (1) applied to its local box)
    const uint32_t cyz = cb / (uint32_t)nb.x, cz = cyz / (uint32_t)nb.y;
    const int b0[3] = {(int)(cb - cyz * nb.x) * nbk[0], (int)(cyz - cz * nb.y) * nbk[1], (int)cz * nbk[2]};
    // The set-up costs as many vector instructions as a hundred points or so do, so what is
    // the same work for several values is done by as many lanes: lane k < 9 takes entry k of the
    // inverse and bound k of the box (a step of 80 models of 131,072 points, 16 grids at 32^3 x 2:
    // 6.22 -> 6.15 ms; hash grids of 8 x 4 levels, 2^20 points: 2.28 -> 2.23 ms; several blocks in turn
    // for one set-up keep more values alive than fit: 6.16 ms at best, 6.8 with one block).
    const float* Gr = a.G + model * a.G_stride + 12 * g;
    const int k9 = min(lane, 8), kr = k9 / 3, kc = k9 - 3 * kr;
    const int c1 = kc == 2 ? 0 : kc + 1, c2 = kc == 0 ? 2 : kc - 1, r1 = kr == 2 ? 0 : kr + 1, r2 = kr == 0 ? 2 : kr - 1;
    const double cof = (double)Gr[4 * c1 + r1] * (double)Gr[4 * c2 + r2] - (double)Gr[4 * c1 + r2] * (double)Gr[4 * c2 + r1];
    const float g0 = Gr[4 * kc];
    const double det = (double)Gg[0] * lane_f64(cof, 0) + (double)Gg[1] * lane_f64(cof, 3) + (double)Gg[2] * lane_f64(cof, 6);
    const float Ak = (float)(cof * recip_f64(det));             // entry k9 of the inverse
    const bool bad = __ballot(!isfinite(Ak)) != 0 || !(fabs(det) > 1e-30);
    int lo[3], hi[3];
    {
      float lm[3], hl[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int e = min(b0[d] + nbk[d], R1);
        const float hc = 0.5f * (float)a.cell;
        lm[d] = -1.f + (float)(b0[d] + e) * hc - Gg[4 * d + 3];   // box centre minus the translation
        hl[d] = (float)(e - b0[d]) * hc;                           // box half-width (local units)
      }
      float wc = 0.f, hw = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const float Ai = __shfl(Ak, 3 * kc + k, 64);
        wc = __builtin_fmaf(Ai, lm[k], wc);
        hw = __builtin_fmaf(fabsf(Ai), hl[k], hw);
      }
      const float f0 = floorf((wc - hw - 1e-4f + 1.f) * (0.5f * kBinsPerAxis));
      const float f1 = floorf((wc + hw + 1e-4f + 1.f) * (0.5f * kBinsPerAxis));
      const int l0 = bad ? 0 : (int)fminf(fmaxf(f0, 0.f), (float)(kBinsPerAxis - 1));
      const int l1 = bad ? kBinsPerAxis - 1 : (int)fminf(fmaxf(f1, 0.f), (float)(kBinsPerAxis - 1));
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        lo[d] = __builtin_amdgcn_readlane(l0, d);
        hi[d] = __builtin_amdgcn_readlane(l1, d);
      }
    }
    constexpr size_t kNB3 = (size_t)kBinsPerAxis * kBinsPerAxis * kBinsPerAxis;
    const float4* P4 = TS == 1 ? a.pts4 + (size_t)model * a.n : a.pts4;
    const float* dY = a.dY + (TS == 1 ? model * a.dY_stride : 0) + (size_t)g * a.dY_grid;
    const uint32_t* start = a.start + (size_t)model * (TS == 1 ? kNB3 + 1 : kNB3);
    const float ht = 0.5f * (float)(a.Rt - 1);
    const float hR = 0.5f * (float)R1;
    // local_box and span_recips: axis kc's lower bound in lanes 0-2, upper bound in 3-5, reciprocal
    // in 6-8 (to scalar registers where the rows are cut: held from here they would be spilled)
    static_assert(kPullNY == kPullNZ, "one width for y and z");
    const int bd = kc == 0 ? b0[0] : kc == 1 ? b0[1] : b0[2], ed = min(bd + (kc == 0 ? nbk[0] : kPullNY), R1);
    const double td = (double)Gr[4 * kc + 3], rec = g0 != 0.f ? recip_f64((double)g0) : 0.0;
    const double box = -1.0 + a.cell * (kr == 0 ? bd : ed) + (kr == 0 ? -1e-4 : 1e-4) - td;
    const double span = kr == 2 ? rec : box;
    const int ny_r = hi[1] - lo[1] + 1, nz_r = hi[2] - lo[2] + 1;
    const int nrows = ny_r * nz_r;
    // the block's cells on an axis: u - ulo in [0, width), cells 0 .. cmax (the grid's last cell
    // includes u = R - 1)
    float ulo[3], cmax[3];
    uint32_t uwid[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const bool last = b0[d] + nbk[d] >= R1;
      ulo[d] = (float)b0[d];
      uwid[d] = __float_as_uint(last ? __builtin_inff() : (float)nbk[d]);
      cmax[d] = (float)(last ? R1 - b0[d] - 1 : nbk[d] - 1);
    }
    const void* Fm = GF16 ? (const void*)((const __half*)a.F + model * a.F_stride)
                          : (const void*)((const float*)a.F + model * a.F_stride);
    struct Cand { float4 q; float dy[C]; bool valid; };
    // lane roles as matrix operands: element e16 of the slots 16 m + 4 k4 + q (q = 0..3 in four
    // instructions)
    const int e16 = lane & 15, k4 = lane >> 4;
    float* ops = sOp[wave];
    const float* rd = ops + e16 * kSlotPitch + 4 * k4;
    auto consume = [&](const Cand& cd) {
      float l[3], u[3], t[3];
      local_coords(Gg, cd.q.x, cd.q.y, cd.q.z, l);
      // the cell decision of Eq. (2): u = fma(l, h, h) is negative below the grid, l <= 1 bounds
      // it above; t = u - (first cell) is exact, and as bits unsigned it is below the width's only
      // for 0 <= t < width (not for a negative value or a NaN)
      bool in = cd.valid && fmaxf(fmaxf(l[0], l[1]), l[2]) <= 1.0f;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        u[d] = __builtin_fmaf(l[d], hR, hR);
        t[d] = u[d] - ulo[d];
        in = in && __float_as_uint(t[d]) < uwid[d];
      }
      float wt = 0.f;
      if constexpr (TS == 2) {
        // the time cell and weight as the 4-D lookup takes them; times outside [-1, 1] add nothing
        const float tq = cd.q.w;
        const float ut = __builtin_fmaf(tq, ht, ht);
        const float ft = fminf(fmaxf(floorf(ut), 0.0f), (float)(a.Rt - 2));
        in = in && tq >= -1.0f && tq <= 1.0f && (int)ft == model;
        wt = ut - ft;
      }
      // a non-finite dL/dy times the zero of a hat function would reach every vertex of the block:
      // such points (none in a healthy run) are added to their cell's corners alone
      float fl[3], w[3];                       // cell in the block and offsets
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        fl[d] = fminf(floorf(t[d]), cmax[d]);
        w[d] = t[d] - fl[d];
      }
      bool wild = false;
#pragma unroll
      for (int c = 0; c < C; ++c) wild = wild || !(fabsf(cd.dy[c]) < __builtin_inff());
      uint64_t wmask = __ballot(in && wild);
      const bool fin = in && !wild;
      const uint64_t mask = __ballot(fin);
      const int v = __popcll(mask);
      if (wmask) {
        do {
          const int k = __builtin_ctzll(wmask);
          wmask &= wmask - 1;
          float uk[3], dk[C];
          for (int d = 0; d < 3; ++d) uk[d] = __shfl(t[d], k, 64);
          for (int c = 0; c < C; ++c) dk[c] = __shfl(cd.dy[c], k, 64);
          const float wk = __shfl(wt, k, 64);
          float wz, wy[4];
          const auto corner = [&](int d, int vtx, float& wgt) {   // weight of a corner of the point's cell
            const float fl = fminf(floorf(uk[d]), cmax[d]), w = uk[d] - fl;
            wgt = (float)vtx == fl ? 1.f - w : w;
            return (float)vtx == fl || (float)vtx == fl + 1.f;
          };
          const bool oz = corner(2, k4, wz);
          bool oy[4];
          for (int r = 0; r < 4; ++r) oy[r] = corner(1, r, wy[r]);
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            const int col = 16 * j + e16, ch = col % CT;
            float wx, d = dk[0];
            const bool ox = corner(0, col / CT, wx);
#pragma unroll
            for (int c = 1; c < C; ++c) d = ch % C == c ? dk[c] : d;
            const float ws = TS == 1 ? 1.f : ch / C ? wk : 1.f - wk;
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (oz && oy[r] && ox) acc[j][r] += ws * (wx * wy[r] * wz) * d;
          }
        } while (wmask);
      }
      if constexpr (DG) {
        if (in) {
          int i0[3];
#pragma unroll
          for (int d = 0; d < 3; ++d) i0[d] = b0[d] + (int)fl[d];
          float val[8][C];
          gather_cell<C, GF16>(Fm, g, s.R, i0, val);
          add_transform_grad<C>(val, w, cd.dy, hR, true, cd.q.x, cd.q.y, cd.q.z, gacc);
        }
      }
      if (v == 0) return;
      const int rk = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
      float* pa = ops + (int)__builtin_fmaf(fl[2], 4.f * kSlotPitch, fl[1] * kSlotPitch) + rk;
      float* pb = ops + (int)__builtin_fmaf(fl[0], (float)(CT * kSlotPitch), 16.f * kSlotPitch) + rk;
      const float wy0 = 1.f - w[1], wz0 = 1.f - w[2], wx0 = 1.f - w[0];
      for (int h = 0; h < v; h += kSlots) {
        const bool mine = fin && (uint32_t)(rk - h) < (uint32_t)kSlots;
        if (mine) {
          pa[0] = wz0 * wy0;
          pa[kSlotPitch] = wz0 * w[1];
          pa[4 * kSlotPitch] = w[2] * wy0;
          pa[5 * kSlotPitch] = w[2] * w[1];
#pragma unroll
          for (int ch = 0; ch < CT; ++ch) {
            float d = cd.dy[ch % C];
            if constexpr (TS == 2) d *= ch / C ? wt : 1.f - wt;
            pb[ch * kSlotPitch] = wx0 * d;
            pb[(CT + ch) * kSlotPitch] = w[0] * d;
          }
        }
        wave_lds_order();
        const int left = v - h;
#pragma unroll
        for (int m = 0; m < kSlots; m += 16) {
          if (m > 0 && m >= left) break;
          const f32x4 av = *(const f32x4*)(rd + m);
          f32x4 bv[NT];
#pragma unroll
          for (int j = 0; j < NT; ++j) bv[j] = *(const f32x4*)(rd + m + 16 * (1 + j) * kSlotPitch);
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < NT; ++j)
              acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[j][q], acc[j], 0, 0, 0);
        }
        wave_lds_order();
        if (mine) {
          pa[0] = 0.f;
          pa[kSlotPitch] = 0.f;
          pa[4 * kSlotPitch] = 0.f;
          pa[5 * kSlotPitch] = 0.f;
#pragma unroll
          for (int ch = 0; ch < 2 * CT; ++ch) pb[ch * kSlotPitch] = 0.f;
        }
        pa -= kSlots;
        pb -= kSlots;
      }
      wave_lds_order();
    };
    // rows (z outer, y inner) kRowBatch at a time; each batch's points are one flat sequence
    for (int rb = 0; rb < nrows; rb += kRowBatch) {
      uint32_t s0 = 0, len = 0;
      const int rr = rb + lane;
      double blo[3], bhi[3], ra[3];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        blo[d] = lane_f64(span, d);
        bhi[d] = lane_f64(span, 3 + d);
        ra[d] = lane_f64(span, 6 + d);
      }
      if (rr < nrows) {
        int x0 = lo[0], x1 = hi[0];
        const int yb = lo[1] + rr % ny_r, zb = lo[2] + rr / ny_r;
        if (bad || row_x_span(Gg, ra, blo, bhi, lo[0], hi[0], yb, zb, x0, x1)) {
          const int row = (zb * kBinsPerAxis + yb) * kBinsPerAxis;
          s0 = start[row + x0];
          len = start[row + x1 + 1] - s0;
        }
      }
      const uint32_t incl = wave_scan_add(len);
      const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
      const uint32_t end = len > 0 ? incl : 0xffffffffu;         // past the row's last candidate
      const uint64_t full = __ballot(len > 0);
      // non-empty rows in order: their offset from flat index to sorted position
      if (len > 0) sDelta[wave][__builtin_amdgcn_mbcnt_hi((uint32_t)(full >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)full, 0u))] = s0 + len - incl;
      constexpr uint32_t kStep = SPLIT ? 256 : 64, kFirst = SPLIT ? 64 : 0;
      Cand ca, cn;
      for (uint32_t wb = 0; wb < total; wb += kWindow) {
        sEnd[wave][lane] = 0;
        wave_lds_order();
        if (end - 1u - wb < kWindow) atomicOr((uint32_t*)sEnd[wave] + ((end - 1u - wb) >> 5), 1u << ((end - 1u) & 31));
        wave_lds_order();
        // candidate f = base + lane lies in the row after those that end before it: the rows that
        // end before the step, plus the row ends among the step's earlier candidates
        auto load = [&](uint32_t base, Cand& cd) {
          const uint64_t em = sEnd[wave][(base - wb) >> 6];
          const uint32_t before = (uint32_t)__popcll(__ballot(end <= base));
          const uint32_t row =
              __builtin_amdgcn_mbcnt_hi((uint32_t)(em >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)em, before));
          const uint32_t f = base + (uint32_t)lane;
          cd.valid = f < total;
          const uint32_t delta = sDelta[wave][row];   // (row is at most kRowBatch, past the last candidate)
          const uint32_t pp = cd.valid ? f + delta : 0u;
          cd.q = P4[pp];
#pragma unroll
          for (int c = 0; c < C; ++c) cd.dy[c] = dY[(size_t)pp * C + c];
        };
        const uint32_t we = min(total, wb + kWindow);
        uint32_t base = wb + kFirst * (uint32_t)wave;
        if (base < we) load(base, ca);
        for (; base < we; base += kStep) {
          if (base + kStep < we) load(base + kStep, cn);
          consume(ca);
          ca = cn;
        }
      }
    }
  }
  float* out = a.CC + (((size_t)model * s.M + g) * nblk_grid + cb) * LAT;
  // D[i][j]: lane j + 16 vz, register vy; column 16 t + j
  auto lat_index = [&](int t, int r) { return ((lane >> 4) * 4 + r) * (VX * CT) + 16 * t + (lane & 15); };
  if constexpr (!SPLIT) {
    if (act) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[lat_index(t, r)] = acc[t][r];
    }
  } else {
    // the four waves' lattices, added in wave order (the operand slots are free by now; a wave
    // writes only its own)
    static_assert(LAT <= (1 + NT) * 16 * kSlotPitch, "a lattice fits a wave's operand slots");
    float* mine = sOp[wave];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) mine[lat_index(t, r)] = acc[t][r];
    __syncthreads();
    if (act) {
      for (int i = threadIdx.x; i < LAT; i += 256) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) sum = add_rounded(sum, sOp[w][i]);
        out[i] = sum;
      }
    }
  }
  if constexpr (DG) {
#pragma unroll
    for (int k = 0; k < 12; ++k) {
      const double t = wave_sum((double)gacc[k]);
      if (lane == 0) sDG[wave][k] = t;
    }
    __syncthreads();
    if (threadIdx.x < 12) {
      const double t = sDG[0][threadIdx.x] + sDG[1][threadIdx.x] + sDG[2][threadIdx.x] + sDG[3][threadIdx.x];
      a.dGpart[(((size_t)model * s.M + g) * groups + grp) * 12 + threadIdx.x] = t;
    }
  }
}

// dF[model][g][v][c] (+)= sum over the cells adjacent to vertex v of their corner sums.
// dF in the paper's order [M][C][R^3] when paper != 0, else channel-last [M][R^3][C].
template <int C>
__global__ void k_cell_to_vertex(Shape s, const float* CC, float* dF, size_t dF_stride, int paper, int accumulate,
                                 const int32_t* active) {
  const int model = blockIdx.z, g = blockIdx.y;
  if (active && !active[model]) return;
  const int R = s.R, R1 = R - 1;
  const int64_t nv = (int64_t)R * R * R, ncell = (int64_t)R1 * R1 * R1;
  const float* cc = CC + ((size_t)model * s.M + g) * 8 * ncell * C;
  for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x) {
    const int vx = (int)(v % R), vy = (int)((v / R) % R), vz = (int)(v / ((int64_t)R * R));
    float sum[C];
#pragma unroll
    for (int c = 0; c < C; ++c) sum[c] = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int cx = vx - (q & 1), cy = vy - ((q >> 1) & 1), cz = vz - (q >> 2);
      if (cx < 0 || cy < 0 || cz < 0 || cx >= R1 || cy >= R1 || cz >= R1) continue;
      const float* src = cc + ((q * ncell + ((int64_t)cz * R1 + cy) * R1 + cx)) * C;   // neighbours read neighbours
#pragma unroll
      for (int c = 0; c < C; ++c) sum[c] += src[c];
    }
    float* dst = dF + model * dF_stride + (paper ? (size_t)g * C * nv + v : ((size_t)g * nv + v) * C);
    const size_t cs = paper ? (size_t)nv : 1;
#pragma unroll
    for (int c = 0; c < C; ++c) dst[c * cs] = accumulate ? dst[c * cs] + sum[c] : sum[c];
  }
}

// Sum over the cell blocks that contain vertex (x, y, z) of their lattice values of channels
// [ch0, ch0 + C) of CT (bl = the grid's first lattice; along each axis a vertex at a block
// boundary belongs to two blocks), in a fixed order.
template <int C, int CT>
__device__ inline void lattice_sum(const float* bl, const PullBlocks& nb, int ch0, int x, int y, int z, float sum[C]) {
  constexpr int VX = pull_vx(C);
  constexpr int nbk[3] = {VX - 1, kPullNY, kPullNZ};
  typedef float vec __attribute__((ext_vector_type(C), aligned(4 * C)));
  const int vc[3] = {x, y, z}, nn[3] = {nb.x, nb.y, nb.z};
  int b0[3], b1[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    // blocks b with 0 <= vc - nbk b <= nbk: the lower one (vc on its upper face) first
    const int q = vc[d] / nbk[d];
    b1[d] = min(q, nn[d] - 1);
    b0[d] = (q * nbk[d] == vc[d] && q > 0) ? q - 1 : b1[d];
  }
#pragma unroll
  for (int c = 0; c < C; ++c) sum[c] = 0.f;
  for (int bz = b0[2]; bz <= b1[2]; ++bz)
    for (int by = b0[1]; by <= b1[1]; ++by)
      for (int bx = b0[0]; bx <= b1[0]; ++bx) {
        const vec v = *(const vec*)(bl + ((((size_t)(bz * nb.y + by) * nb.x + bx) * 16 + (vc[2] - nbk[2] * bz) * 4 +
                                          (vc[1] - nbk[1] * by)) * VX + (vc[0] - nbk[0] * bx)) * CT + ch0);
        if constexpr (C == 1) sum[0] += v[0];
        else {
#pragma unroll
          for (int c = 0; c < C; ++c) sum[c] += v[c];
        }
      }
}

// dF[model][g][v][c] (+)= the lattice sums of every vertex (the output of k_block_pull).  dF
// layout as for k_cell_to_vertex.
template <int C>
__global__ void k_block_to_vertex(Shape s, const float* BL, float* dF, size_t dF_stride, int paper, int accumulate,
                                  const int32_t* active) {
  const int model = blockIdx.z, g = blockIdx.y;
  if (active && !active[model]) return;
  const uint32_t R = s.R, nv = R * R * R;    // (a grid holds fewer than 2^31 values)
  const PullBlocks nb = pull_blocks(R, C);
  const float* bl = BL + ((size_t)model * s.M + g) * nb.total() * pull_lat(C) * C;
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t yz = v / R, z = yz / R;
    float sum[C];
    lattice_sum<C, C>(bl, nb, 0, (int)(v - yz * R), (int)(yz - z * R), (int)z, sum);
    float* dst = dF + model * dF_stride + (paper ? (size_t)g * C * nv + v : ((size_t)g * nv + v) * C);
    const size_t cs = paper ? (size_t)nv : 1;
#pragma unroll
    for (int c = 0; c < C; ++c) dst[c * cs] = accumulate ? dst[c * cs] + sum[c] : sum[c];
  }
}

// 4-D grids: dF[g][t][v][c] (+)= the slice-0 lattice sums of time cell t and the slice-1 sums
// of time cell t - 1 (the output of the TS = 2 pass); a fixed order.  dF in the paper's order
// [M][C][Rt][R^3] when paper != 0, else channel-last [M][Rt][R^3][C].
template <int C>
__global__ void k_block_to_vertex_time(Shape s, int Rt, const float* BL, float* dF, int paper, int accumulate) {
  const int g = blockIdx.y, tv = blockIdx.z;
  const uint32_t R = s.R, nv = R * R * R;
  const PullBlocks nb = pull_blocks(R, C);
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t yz = v / R, z = yz / R;
    float sum[C];
#pragma unroll
    for (int c = 0; c < C; ++c) sum[c] = 0.f;
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
      const int tc = tv - sl;
      if (tc < 0 || tc > Rt - 2) continue;
      const float* bl = BL + ((size_t)tc * s.M + g) * nb.total() * pull_lat(C) * C * 2;
      float part[C];
      lattice_sum<C, 2 * C>(bl, nb, C * sl, (int)(v - yz * R), (int)(yz - z * R), (int)z, part);
#pragma unroll
      for (int c = 0; c < C; ++c) sum[c] += part[c];
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      float* dst = dF + (paper ? ((size_t)(g * C + c) * Rt + tv) * nv + v : (((size_t)g * Rt + tv) * nv + v) * C + c);
      *dst = accumulate ? *dst + sum[c] : sum[c];
    }
  }
}

// dG[model][g][k] (+)= sum over the cb per-block partials of grid g: one workgroup per (grid,
// model); thread t sums blocks t, t + 256, ... in order, then a fixed tree over the threads.
// dG rows per transform: grows (3, or 4 with row 3 written as 0).
__global__ void __launch_bounds__(256) k_reduce_cell_dG(const double* part, int M, int cb, double* dG,
                                                        size_t dG_stride, int grows, int accumulate,
                                                        const int32_t* active) {
  __shared__ double sp[256][13];
  const int g = blockIdx.x, model = blockIdx.y;
  if (active && !active[model]) return;
  const double* P = part + ((size_t)model * M + g) * cb * 12;
  double acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0;
  for (int b = threadIdx.x; b < cb; b += blockDim.x)
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] += P[(size_t)b * 12 + k];
#pragma unroll
  for (int k = 0; k < 12; ++k) sp[threadIdx.x][k] = acc[k];
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (threadIdx.x < w)
#pragma unroll
      for (int k = 0; k < 12; ++k) sp[threadIdx.x][k] += sp[threadIdx.x + w][k];
    __syncthreads();
  }
  if (threadIdx.x < 12) {
    double* o = dG + model * dG_stride + 4 * grows * g + threadIdx.x;
    *o = accumulate ? *o + sp[0][threadIdx.x] : sp[0][threadIdx.x];
  } else if (grows == 4 && threadIdx.x < 16 && !accumulate) {
    dG[model * dG_stride + 4 * grows * g + threadIdx.x] = 0.0;
  }
}

}  // namespace apmg
