// Global-query inference over a domain decomposition (Sec. 5.3).  Each global
// point is hashed to its brick, and the points are ordered by brick and, inside a
// brick, by spatial bin (a stable radix sort), so that one launch of the forward
// tile kernel evaluates every brick's points with its own model (block row =
// brick, a contiguous segment of the order): it reads each point and writes its
// output through the order's permutation and maps the point into its brick's
// local frame itself.

namespace apmg {

// Brick of global point (x, y, z): the voxel coordinate u = fma(p, h, h),
// h = (n-1)/2, selects the base brick holding floor(u), clamped to the grid.
__device__ inline int brick_of(const apmg_brick_table& t, const float p[3]) {
  int idx[3];
  for (int d = 0; d < 3; ++d) {
    const float h = 0.5f * (float)(t.vol[d] - 1);
    float u = __builtin_fmaf(p[d], h, h);
    if (!(fabsf(u) <= 3.0e38f)) u = 0.f;  // a non-finite coordinate goes to brick 0 on that axis
    const float fl = fminf(fmaxf(floorf(u), 0.f), (float)t.vol[d]);
    const int k = (int)fl / t.B;
    idx[d] = k < t.dims[d] - 1 ? k : t.dims[d] - 1;
  }
  return idx[0] + t.dims[0] * (idx[1] + t.dims[1] * idx[2]);
}

// Sort key of a global point: its brick, followed by bits of its bin inside the brick (x fastest:
// bits[0] of x, bits[1] of y, bits[2] of z; none where the order does not pay).  The bin only orders the work
// -- a tile's points then share grid cells in cache -- so it may round as it likes.  The point
// is also written as one 16-byte record: read through the permutation, a record is one cache line
// where the three coordinate rows are three (4.0 M points, 80 models: 0.92 -> 0.87 ms for the whole query).
struct DdKey {
  apmg_brick_table t; const apmg_brick* bricks; int3 bits; const float* pts; int64_t ld; float4* rec;
  __device__ inline uint32_t operator()(int, int64_t i) const {
    const float p[3] = {pts[i], pts[ld + i], pts[2 * ld + i]};
    rec[i] = make_float4(p[0], p[1], p[2], 0.f);
    uint32_t key = (uint32_t)brick_of(t, p);
    const int nbits[3] = {bits.x, bits.y, bits.z};
    if (nbits[0] > 0) {
      const apmg_brick br = bricks[key];
#pragma unroll
      for (int d = 2; d >= 0; --d) {
        const float h = 0.5f * (float)(t.vol[d] - 1), e0 = (float)br.e0[d], span = (float)(br.e1[d] - br.e0[d]);
        const float top = (float)((1 << nbits[d]) - 1);
        const float b = (__builtin_fmaf(p[d], h, h) - e0) * __frcp_rn(span + 1.f) * (top + 1.f);
        key = (key << nbits[d]) | (uint32_t)fminf(fmaxf(b, 0.f), top);   // (NaN -> 0)
      }
    }
    return key;
  }
};

// start[b] = first position whose key >> shift is >= b, b in [0, nseg]; binary search.
__global__ void k_seg_starts(const uint32_t* keys, int64_t n, int shift, int nseg, uint32_t* start) {
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b <= nseg; b += gridDim.x * blockDim.x) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      if ((keys[mid] >> shift) < (uint32_t)b) lo = mid + 1; else hi = mid;
    }
    start[b] = (uint32_t)lo;
  }
}

}  // namespace apmg
