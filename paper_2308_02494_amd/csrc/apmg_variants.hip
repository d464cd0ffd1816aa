// Adjoint of the two encoder variants of Sec. 9 (a hash grid inside each adaptive grid; 4-D
// grids with a time axis) with respect to their tables / grids and the transforms.
//
// The forward and the MLP adjoint are the tile kernels (k_forward, k_adjoint) instantiated
// with the variant's lookup (enc_tap); k_adjoint stores dL/dy per (feature grid, point) of the
// spatially sorted points.
//
// Table gradient of a hash level: a level of N cells per axis is a dense grid of (N + 1)^3
// vertices until its vertices are mapped to entries, so its vertex sums come from the block
// gather of the dense grids (k_block_pull), and the vertices of an entry are then added
// (k_lattice_to_table, k_lattice_to_hash): no atomics, a fixed order.  Levels with many more
// vertices than the batch has points (or a table smaller than a row of vertices), and all levels
// of a small batch, take the scatter instead (k_enc_scatter): w_q dL/dy_c added to the corner entries with float atomics,
// where each wave first sums the runs of lanes with the same cell and only the run's first
// lane issues the atomics; those sums are reproducible to rounding only.  The 4-D grids take
// the block gather per time cell, or the scatter beyond 513 time vertices.  The transform
// gradient through the interpolation weights is reduced per block in float64, in a fixed
// order (k_enc_transform_grad).

namespace apmg {

struct EncScatterArgs {
  Shape s;
  EncArgs enc;
  const float* G;          // [M / L][12]
  const float* F;          // hash: tables [M][T][C]; time: channel-last [M][Rt][R^3][C]
  const float* pts; int64_t ld; int64_t n;
  const float* tau;        // time: [n] time of each point
  const float* dY;         // [M][n][C], dL/dy per feature grid (M feature grids)
  float* dF;               // scatter: same layout as F (channel-last for time), accumulated
  int nlev, lev[kMaxLevels];   // scatter: block row y is level lev[y % nlev] of adaptive grid y / nlev
  double* dGpart;          // transform gradient: [M][nbx][12]
  int nbx;                 // point blocks per feature grid, of 256 tgp points
  int tgp;
};

// dl_d = sum_c dy_c d(trilinear_c)/dw_d for corner values val and offsets w.
template <int C>
__device__ inline void trilerp_dw(const float val[8][C], const float w[3], const float dy[C], float dl[3]) {
#pragma unroll
  for (int d = 0; d < 3; ++d) dl[d] = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float wx = (q & 1) ? w[0] : 1.f - w[0], wy = (q & 2) ? w[1] : 1.f - w[1], wz = (q & 4) ? w[2] : 1.f - w[2];
    const float sx = (q & 1) ? 1.f : -1.f, sy = (q & 2) ? 1.f : -1.f, sz = (q & 4) ? 1.f : -1.f;
    float gq = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) gq = __builtin_fmaf(val[q][c], dy[c], gq);
    dl[0] = __builtin_fmaf(gq * sx, wy * wz, dl[0]);
    dl[1] = __builtin_fmaf(gq * sy, wx * wz, dl[1]);
    dl[2] = __builtin_fmaf(gq * sz, wx * wy, dl[2]);
  }
}

__device__ inline float tri_weight(int q, const float w[3]) {
  return ((q & 1) ? w[0] : 1.f - w[0]) * ((q & 2) ? w[1] : 1.f - w[1]) * ((q & 4) ? w[2] : 1.f - w[2]);
}

// Runs of consecutive lanes with the same key (the points are spatially sorted, so
// neighbouring lanes mostly share a cell): seg = the run's first lane; nxt[k] = lane
// + 2^k is in the same run.  A segmented suffix sum over the run then leaves each run's
// total in its first lane, which alone issues the atomics.
struct WaveRuns {
  bool head;
  bool nxt[6];
};
__device__ inline WaveRuns wave_runs(uint64_t key, int lane) {
  WaveRuns r;
  const uint32_t klo = (uint32_t)key, khi = (uint32_t)(key >> 32);
  const uint32_t plo = __shfl_up(klo, 1, 64), phi = __shfl_up(khi, 1, 64);
  r.head = lane == 0 || plo != klo || phi != khi;
  int seg = r.head ? lane : 0;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(seg, o, 64);
    if (lane >= o) seg = max(seg, t);
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int o = 1 << k;
    const int t = __shfl_down(seg, o, 64);
    r.nxt[k] = lane + o < 64 && t == seg;
  }
  return r;
}
__device__ inline float run_sum(float v, const WaveRuns& r) {
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const float t = __shfl_down(v, 1 << k, 64);
    v += r.nxt[k] ? t : 0.f;
  }
  return v;
}

// One thread per (point, feature grid): 256 points per block.
template <int C, int ENC>
__global__ void __launch_bounds__(256) k_enc_scatter(EncScatterArgs a) {
  const Shape s = a.s;
  const int g = (int)(blockIdx.y / a.nlev) * s.L + a.lev[blockIdx.y % a.nlev];
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = p < a.n;
  float x = 0.f, y = 0.f, z = 0.f, tq = 0.f;
  if (valid) { x = a.pts[p]; y = a.pts[a.ld + p]; z = a.pts[2 * a.ld + p]; }
  if constexpr (ENC == kEncTime) tq = valid ? a.tau[p] : 0.f;
  float dy[C];
#pragma unroll
  for (int c = 0; c < C; ++c) dy[c] = valid ? a.dY[((size_t)g * a.n + p) * C + c] : 0.f;
  // the cell of this lane's point (the same float32 decision as the lookup)
  const int gt = g / s.L, N = ENC == kEncHash ? enc_level_res(a.enc, g - gt * s.L) : s.R - 1;
  float l[3], w[3];
  int i0[3];
  local_coords(a.G + 12 * gt, x, y, z, l);
  bool in = cell_of(l, 0.5f * (float)N, N + 1, i0, w) && valid;
  const int lane = threadIdx.x & 63;
  if constexpr (ENC == kEncHash) {
    const uint64_t key = in ? ((uint64_t)i0[2] << 40 | (uint64_t)i0[1] << 20 | (uint64_t)i0[0]) : ~0ull - lane;
    const WaveRuns rn = wave_runs(key, lane);
    const uint32_t n1 = (uint32_t)N + 1u;
    const bool dense = (uint64_t)n1 * n1 * n1 <= (uint64_t)a.enc.tmask + 1u;
    float* base = a.dF + (size_t)g * ((size_t)a.enc.tmask + 1u) * C;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float wq = in ? tri_weight(q, w) : 0.f;
      float v[C];
#pragma unroll
      for (int c = 0; c < C; ++c) v[c] = run_sum(wq * dy[c], rn);
      if (in && rn.head) {
        const uint32_t ent = hash_entry((uint32_t)i0[0] + (q & 1), (uint32_t)i0[1] + ((q >> 1) & 1),
                                        (uint32_t)i0[2] + (q >> 2), n1, dense, a.enc.tmask);
#pragma unroll
        for (int c = 0; c < C; ++c) unsafeAtomicAdd(base + (size_t)ent * C + c, v[c]);
      }
    }
  } else {
    const float ht = 0.5f * (float)(a.enc.Rt - 1);
    const float ut = __builtin_fmaf(tq, ht, ht);
    const float ft = fminf(fmaxf(floorf(ut), 0.0f), (float)(a.enc.Rt - 2));
    const int t0 = (int)ft;
    const float wt = ut - ft;
    in = in && tq >= -1.0f && tq <= 1.0f;
    const uint32_t R = (uint32_t)s.R, RC = R * C, RRC = R * R * C;
    const uint64_t key = in ? ((((uint64_t)t0 * R + i0[2]) * R + i0[1]) * R + i0[0]) : ~0ull - lane;
    const WaveRuns rn = wave_runs(key, lane);
    const uint32_t cb = in ? ((uint32_t)i0[2] * R + i0[1]) * RC + (uint32_t)i0[0] * C : 0u;
#pragma unroll
    for (int sl = 0; sl < 2; ++sl) {
      const float ws = sl ? wt : 1.f - wt;
      float* base = a.dF + (((size_t)g * a.enc.Rt + (in ? t0 : 0) + sl) * R * R * R) * C;
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float wq = in ? ws * tri_weight(q, w) : 0.f;
        const uint32_t o = cb + (q & 1) * C + ((q >> 1) & 1) * RC + (q >> 2) * RRC;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const float v = run_sum(wq * dy[c], rn);
          if (in && rn.head) unsafeAtomicAdd(base + o + c, v);
        }
      }
    }
  }
}

// Table gradient of one level whose vertices have an entry each: entry v of adaptive grid gt
// += the lattice sums of vertex v (tables at gt * table_stride floats).
template <int C>
__global__ void k_lattice_to_table(int N, const float* BL, float* dF, size_t table_stride) {
  const int gt = blockIdx.y;
  const uint32_t n1 = N + 1, nv = n1 * n1 * n1;
  const PullBlocks nb = pull_blocks((int)n1, C);
  const float* bl = BL + gt * nb.total() * pull_lat(C) * C;
  for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
    const uint32_t yz = v / n1, z = yz / n1;
    float sum[C];
    lattice_sum<C, C>(bl, nb, 0, (int)(v - yz * n1), (int)(yz - z * n1), (int)z, sum);
    float* dst = dF + gt * table_stride + (size_t)v * C;
#pragma unroll
    for (int c = 0; c < C; ++c) dst[c] += sum[c];
  }
}

// Table gradient of a hashed level: entry e += the lattice sums of every vertex that hashes to
// e.  The hash is x XOR h(y, z) in its low bits, so a row of vertices (y, z) with N + 1 <= B = 64
// NB vertices falls into one aligned run of B entries, entry e of the run holding vertex x =
// (e XOR h) mod B.  A workgroup owns one run: each of its four waves scans its share of the
// rows 64 at a time (h of a row per lane, one ballot finds the rows of this run) and adds the
// matching rows in order, lane i holding the entries i, i + 64, ... of the run; the four waves'
// sums are then added in order.  No atomics, and every vertex is read once.
template <int C, int NB>
__global__ void __launch_bounds__(256) k_lattice_to_hash(int N, uint32_t tmask, const float* BL, float* dF,
                                                         size_t table_stride) {
  constexpr int VX = pull_vx(C), NX = VX - 1;
  constexpr uint32_t B = 64 * NB;
  typedef float vec __attribute__((ext_vector_type(C), aligned(4 * C)));
  __shared__ float sSum[4][B * C];
  const int gt = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n1 = N + 1, rows = n1 * n1, run = blockIdx.x * B;
  const PullBlocks nb = pull_blocks((int)n1, C);
  const float* bl = BL + gt * nb.total() * pull_lat(C) * C;
  float acc[NB][C];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int c = 0; c < C; ++c) acc[i][c] = 0.f;
  for (uint32_t r0 = 64u * wave; r0 < rows; r0 += 256) {
    const uint32_t r = r0 + lane, z = r / n1, y = r - z * n1;
    const uint32_t h = (y * 2654435761u) ^ (z * 805459861u);
    uint64_t m = __ballot(r < rows && ((h & tmask) & ~(B - 1u)) == run);
    while (m) {
      const int k = __builtin_ctzll(m);
      m &= m - 1;
      const uint32_t hk = __builtin_amdgcn_readlane((int)h, k);
      const int zk = __builtin_amdgcn_readlane((int)z, k), yk = __builtin_amdgcn_readlane((int)y, k);
      // the one or two blocks along y and z that hold the row (the lower one first)
      const int qy = yk / kPullNY, qz = zk / kPullNZ;
      const int by1 = min(qy, nb.y - 1), by0 = (qy * kPullNY == yk && qy > 0) ? qy - 1 : by1;
      const int bz1 = min(qz, nb.z - 1), bz0 = (qz * kPullNZ == zk && qz > 0) ? qz - 1 : bz1;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const uint32_t x = ((uint32_t)(lane + 64 * i) ^ hk) & (B - 1u);
        if (x > (uint32_t)N) continue;
        const int qx = (int)x / NX;
        const int bx1 = min(qx, nb.x - 1), bx0 = (qx * NX == (int)x && qx > 0) ? qx - 1 : bx1;
        for (int bz = bz0; bz <= bz1; ++bz)
          for (int by = by0; by <= by1; ++by)
            for (int bx = bx0; bx <= bx1; ++bx) {
              const vec v = *(const vec*)(bl + ((((size_t)(bz * nb.y + by) * nb.x + bx) * 16 + (zk - kPullNZ * bz) * 4 +
                                                (yk - kPullNY * by)) * VX + ((int)x - NX * bx)) * C);
#pragma unroll
              for (int c = 0; c < C; ++c) acc[i][c] += v[c];
            }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int c = 0; c < C; ++c) sSum[wave][(lane + 64 * i) * C + c] = acc[i][c];
  __syncthreads();
  float* dst = dF + gt * table_stride + (size_t)run * C;
  for (uint32_t i = threadIdx.x; i < B * C; i += 256)
    dst[i] += ((sSum[0][i] + sSum[1][i]) + sSum[2][i]) + sSum[3][i];
}

// The transform gradient through the interpolation weights: per feature grid, sums over the
// points of (dl_d) x^T and dl_d, in float64.  Several points per thread (a.tgp), so the wave
// reduction of the 12 sums (a butterfly of float64 shuffles, several times the work of a
// point) is paid once per block and not once per point.
constexpr int kTgPoints = 16;              // at most
// Points per thread: 16 once that leaves four blocks per compute unit, fewer for smaller batches, whose
// blocks would run 16 points in a row with most of the device idle (8 grids at 64^3, 4096 points, the
// transform gradient alone: 166 us with 16, 122 with one; 65,536 points: 142 and 129).
inline int tg_points(int64_t n, int grids) {
  return (int)std::max<int64_t>(1, std::min<int64_t>(kTgPoints, n * grids / (256 * 1024)));
}
inline int tg_blocks(int64_t n, int grids) {
  const int64_t per = 256 * tg_points(n, grids);
  return (int)std::max<int64_t>(1, (n + per - 1) / per);
}
template <int C, int ENC>
__global__ void __launch_bounds__(256) k_enc_transform_grad(EncScatterArgs a) {
  __shared__ double sred[4][12];
  const Shape s = a.s;
  const int g = blockIdx.y, bx = blockIdx.x, gt = g / s.L;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float hR = 0.5f * (float)(s.R - 1);
  const float sc = ENC == kEncHash ? 0.5f * (float)enc_level_res(a.enc, g - gt * s.L) : hR;
  double acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0;
  const int64_t p0 = (int64_t)bx * (256 * a.tgp);
  for (int64_t p = p0 + threadIdx.x; p < min(a.n, p0 + 256 * a.tgp); p += 256) {
    const float x = a.pts[p], y = a.pts[a.ld + p], z = a.pts[2 * a.ld + p];
    const float tq = ENC == kEncTime ? a.tau[p] : 0.f;
    float dy[C];
#pragma unroll
    for (int c = 0; c < C; ++c) dy[c] = a.dY[((size_t)g * a.n + p) * C + c];
    GridTap<C, ENC> t;
    enc_tap<C, false, ENC>(s, a.G, GridSrc<ENC>(s, a.F, 4), a.enc, g, x, y, z, tq, true, hR, t);
    if (!t.in) continue;
    float dl[3];
    if constexpr (ENC == kEncHash) {
      trilerp_dw<C>(t.val, t.w, dy, dl);
    } else {
      float d0[3], d1[3];
      trilerp_dw<C>(t.va, t.w, dy, d0);
      trilerp_dw<C>(t.vb, t.w, dy, d1);
#pragma unroll
      for (int d = 0; d < 3; ++d) dl[d] = (1.f - t.wt) * d0[d] + t.wt * d1[d];
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const double d = (double)(dl[r] * sc);
      acc[4 * r] += d * (double)x;
      acc[4 * r + 1] += d * (double)y;
      acc[4 * r + 2] += d * (double)z;
      acc[4 * r + 3] += d;
    }
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    const double v = wave_sum(acc[k]);
    if (lane == 0) sred[wave][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    const double v = sred[0][threadIdx.x] + sred[1][threadIdx.x] + sred[2][threadIdx.x] + sred[3][threadIdx.x];
    a.dGpart[((size_t)g * a.nbx + bx) * 12 + threadIdx.x] = v;
  }
}

// dst[j] = src[perm[j]] (a per-point array in spatially sorted order).
__global__ void k_gather_f32(const float* __restrict__ src, const uint32_t* __restrict__ perm, int64_t n,
                             float* __restrict__ dst) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
    dst[j] = src[perm[j]];
}

// 4-D grids: the time cell of spatially sorted position j (the float32 decision of the lookup;
// outside or NaN times -> 0), the key of the further sort by time.
struct TimeKey {
  const float* tau; const uint32_t* perm; int Rt;
  __device__ inline uint32_t operator()(int, int64_t j) const {
    const float ht = 0.5f * (float)(Rt - 1), t = tau[perm[j]];
    const float ft = fminf(fmaxf(floorf(__builtin_fmaf(t, ht, ht)), 0.0f), (float)(Rt - 2));
    return (t >= -1.0f && t <= 1.0f) ? (uint32_t)ft : 0u;
  }
};

// The points, dL/df and times in (time cell, spatial bin) order: position j takes spatially
// sorted position q = perm2[j] (original point perm[q]); also as (x, y, z, t) records.  perm2 NULL
// (one time cell: the spatial order is that order already): the times and the records alone.
__global__ void k_time_permute(const float* __restrict__ spts, const float* __restrict__ sf,
                               const float* __restrict__ tau, const uint32_t* __restrict__ perm,
                               const uint32_t* __restrict__ perm2, int64_t n, float* __restrict__ pts2,
                               float* __restrict__ f2, float* __restrict__ tau2, float4* __restrict__ rec) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t q = perm2 ? perm2[j] : (uint32_t)j;
    const float x = spts[q], y = spts[n + q], z = spts[2 * n + q], t = tau[perm[q]];
    tau2[j] = t;
    rec[j] = make_float4(x, y, z, t);
    if (!perm2) continue;
    pts2[j] = x;
    pts2[n + j] = y;
    pts2[2 * n + j] = z;
    f2[j] = sf[q];
  }
}

// start[k] for k in [0, (Rt - 1) NB^3]: the first position of the (time cell, bin) order whose
// combined key tc NB^3 + bin is >= k (as k_bin_starts over the combined keys: time keys
// tkey[j] of the sorted order, bin keys bkey[pos[j]] of the spatial order it was taken from).
__global__ void k_time_bin_starts(const uint32_t* __restrict__ tkey, const uint32_t* __restrict__ bkey,
                                  const uint32_t* __restrict__ pos, int64_t n, int Rt, uint32_t* __restrict__ start) {
  const uint32_t nb3 = (uint32_t)kBinsPerAxis * kBinsPerAxis * kBinsPerAxis;
  const uint32_t nkeys = (uint32_t)(Rt - 1) * nb3;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i <= n; i += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t lo = i == 0 ? 0u : tkey[i - 1] * nb3 + bkey[pos[i - 1]] + 1u;
    const uint32_t hi = i == n ? nkeys : tkey[i] * nb3 + bkey[pos[i]];
    for (uint32_t b = lo; b <= hi; ++b) start[b] = (uint32_t)i;
  }
}

// Channel-last [nm][V][C] -> the paper's order [nm][C][V], added into dst when accumulate.
template <int C>
__global__ void k_cl_to_paper(int64_t nm, int64_t V, const float* __restrict__ src, float* __restrict__ dst,
                              int accumulate) {
  const int64_t total = nm * V;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t g = i / V, v = i - g * V;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      float* d = dst + (g * C + c) * V + v;
      *d = accumulate ? *d + src[i * C + c] : src[i * C + c];
    }
  }
}

// rows: adaptive grids times levels taken
hipError_t launch_enc_scatter(const EncScatterArgs& a, int enc, int rows, hipStream_t st) {
  const dim3 grid((unsigned)((a.n + 255) / 256), (unsigned)rows);
  if (a.s.C != 2) return hipErrorInvalidValue;
  if (enc == kEncHash) hipLaunchKernelGGL((k_enc_scatter<2, kEncHash>), grid, dim3(256), 0, st, a);
  else if (enc == kEncTime) hipLaunchKernelGGL((k_enc_scatter<2, kEncTime>), grid, dim3(256), 0, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}
hipError_t launch_enc_transform_grad(const EncScatterArgs& a, int enc, hipStream_t st) {
  const dim3 grid((unsigned)a.nbx, (unsigned)a.s.M);
  if (a.s.C != 2) return hipErrorInvalidValue;
  if (enc == kEncHash) hipLaunchKernelGGL((k_enc_transform_grad<2, kEncHash>), grid, dim3(256), 0, st, a);
  else if (enc == kEncTime) hipLaunchKernelGGL((k_enc_transform_grad<2, kEncTime>), grid, dim3(256), 0, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// A hash level takes the block gather (k_block_pull + k_lattice_to_table / k_lattice_to_hash) while
// its vertices are at most four per point: its lattices then stay small next to dL/dy and a block of
// 63 cells has points enough to pay for finding its candidates.  (A block stores 1 KiB for up to 63
// cells: N = 128 at four vertices a point takes 67 bytes per point and grid, N = 8 about 100.)
// A hashed level's rows also have to fit one aligned run of entries of the table, and a
// workgroup's registers (at most 1024 entries a run).  Measured at 2^20 points, 8 grids: the
// gather and fold of N = 16 / 32 / 64 / 128 take 0.13 / 0.10 / 0.17 / 0.54 ms, the atomics 2.5 ms per level.
// Below kHashPullMin points the two launches a level are the cost (20 and 5 us each) and the
// atomics of all levels, one launch, the better: 4 grids of 3 levels, dL/dtheta alone, 1024 points
// 183 us with the atomics and 222 with the gather; 4096 points 162 and 160; 16384 points 285 and 155.
constexpr int64_t kHashPullMin = 4096;
inline int hash_run_log2(int N) {   // log2 of B, the power of two >= N + 1 and >= 64
  int b = 6;
  while ((1 << b) < N + 1) ++b;
  return b;
}
inline bool hash_level_dense(const EncArgs& e, int N) {
  return (uint64_t)(N + 1) * (N + 1) * (N + 1) <= (uint64_t)e.tmask + 1u;
}
inline bool hash_level_pull(const EncArgs& e, int N, int64_t n) {
  if (n < kHashPullMin || (double)(N + 1) * (N + 1) * (N + 1) > 4.0 * (double)n) return false;
  const int b = hash_run_log2(N);
  return hash_level_dense(e, N) || (b <= 10 && (1u << b) <= e.tmask + 1u);
}
hipError_t launch_lattice_to_entries(const EncArgs& e, int N, int mt, const float* lat, float* dF, size_t table_stride,
                                     hipStream_t st) {
  if (hash_level_dense(e, N)) {
    const int64_t nv = (int64_t)(N + 1) * (N + 1) * (N + 1);
    hipLaunchKernelGGL(k_lattice_to_table<2>, dim3((unsigned)std::min<int64_t>((nv + 255) / 256, 1024), mt), dim3(256), 0,
                       st, N, lat, dF, table_stride);
    return hipGetLastError();
  }
  const int b = hash_run_log2(N);
  const dim3 grid((e.tmask + 1u) >> b, mt);
  if (b == 6) hipLaunchKernelGGL((k_lattice_to_hash<2, 1>), grid, dim3(256), 0, st, N, e.tmask, lat, dF, table_stride);
  else if (b == 7) hipLaunchKernelGGL((k_lattice_to_hash<2, 2>), grid, dim3(256), 0, st, N, e.tmask, lat, dF, table_stride);
  else if (b == 8) hipLaunchKernelGGL((k_lattice_to_hash<2, 4>), grid, dim3(256), 0, st, N, e.tmask, lat, dF, table_stride);
  else if (b == 9) hipLaunchKernelGGL((k_lattice_to_hash<2, 8>), grid, dim3(256), 0, st, N, e.tmask, lat, dF, table_stride);
  else if (b == 10) hipLaunchKernelGGL((k_lattice_to_hash<2, 16>), grid, dim3(256), 0, st, N, e.tmask, lat, dF, table_stride);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// The tile kernels of the variants (C = 2, H = 64): forward with the weights in LDS, and the
// tiled adjoint with the waves per block of the dense shapes.
hipError_t launch_enc_forward(const TileArgs& a, int enc, bool bf, dim3 grid, size_t shmem, hipStream_t st) {
  if (a.s.C != 2 || a.s.H != 64 || fwd_weight_bytes(a.s, bf) > kFwdWeightLdsMax) return hipErrorInvalidValue;
#define APMG_EF(E)                                                                                \
  if (bf) hipLaunchKernelGGL((k_forward<2, 64, false, true, true, E>), grid, dim3(kBlock), shmem, st, a); \
  else hipLaunchKernelGGL((k_forward<2, 64, false, false, true, E>), grid, dim3(kBlock), shmem, st, a);
  if (enc == kEncHash) { APMG_EF(kEncHash) }
  else if (enc == kEncTime) { APMG_EF(kEncTime) }
  else return hipErrorInvalidValue;
#undef APMG_EF
  return hipGetLastError();
}

hipError_t launch_enc_adjoint(const TileArgs& a, int enc, bool bf, dim3 grid, hipStream_t st) {
  if (a.s.C != 2 || !adjoint_applies(a.s)) return hipErrorInvalidValue;
  const int nw = adjoint_waves(0, bf);
  const size_t shmem = adjoint_lds_bytes(a.s, bf, nw);
  // 32 feature grids of 2 (64 features): the adjoint compiled for that shape
  const bool kf32 = a.s.M == 32;
#define APMG_EA(E, KF_)                                                                                     \
  if (bf) hipLaunchKernelGGL((k_adjoint<2, false, true, 4, E, KF_>), grid, dim3(4 * kWave), shmem, st, a);  \
  else hipLaunchKernelGGL((k_adjoint<2, false, false, 8, E, KF_>), grid, dim3(8 * kWave), shmem, st, a);
  if (enc == kEncHash) { if (kf32) { APMG_EA(kEncHash, 32) } else { APMG_EA(kEncHash, 0) } }
  else if (enc == kEncTime) { if (kf32) { APMG_EA(kEncTime, 32) } else { APMG_EA(kEncTime, 0) } }
  else return hipErrorInvalidValue;
#undef APMG_EA
  return hipGetLastError();
}

}  // namespace apmg
