// Acceleration-structure build: activity and bounds of the Gaussians, Z-order
// (Morton) keys, a stable sort, the per-Gaussian records computed in Z order,
// and a Karras LBVH whose node boxes come from range unions over a segment
// tree of the leaf boxes.  Every size follows from N on the host; the number
// of active Gaussians stays on the device, so the whole build is asynchronous.
// Bound by memory: 3.1 ms at 5M Gaussians (0.8 of them the sort), 0.71 ms at
// 1M, and by nine launches (two more with lobes) up to 4096 (0.09 ms); with
// records made in user order and gathered, one scanning workgroup, a launch for
// each tree level and both forms of the 4-wide nodes it was 7.2, 1.54 and 0.22
// ms.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace rgx {

__global__ void k_build_init(uint32_t *bounds, int32_t *counters) {
  int t = threadIdx.x;
  if (t < 3) bounds[t] = 0xffffffffu;        // min
  else if (t < 6) bounds[t] = 0u;            // max
  if (t < 8) counters[t] = 0;
}

// One Gaussian's parameters; `ok` says whether it is active: a finite mean,
// finite scales above zero, a quaternion of finite non-zero norm and a finite
// density above sigma_eps.
struct Params {
  float mu[3], s[3], q[4], sig, qn2;
  bool ok;
};
__device__ __forceinline__ Params load_params(int64_t i, const float *__restrict__ means,
                                              const float *__restrict__ log_scales,
                                              const float *__restrict__ quats,
                                              const float *__restrict__ density, float sigma_eps) {
  Params p;
  float ls[3];
  for (int k = 0; k < 3; k++) { p.mu[k] = means[3 * i + k]; ls[k] = log_scales[3 * i + k]; }
  for (int k = 0; k < 4; k++) p.q[k] = quats[4 * i + k];
  p.sig = density[i];
  p.qn2 = p.q[0] * p.q[0] + p.q[1] * p.q[1] + p.q[2] * p.q[2] + p.q[3] * p.q[3];
  p.ok = isfinite(p.mu[0]) && isfinite(p.mu[1]) && isfinite(p.mu[2]) && isfinite(ls[0]) &&
         isfinite(ls[1]) && isfinite(ls[2]) && isfinite(p.qn2) && p.qn2 > 0.0f && isfinite(p.sig) &&
         p.sig > sigma_eps;
  for (int k = 0; k < 3; k++) {
    p.s[k] = expf(ls[k]);
    p.ok = p.ok && p.s[k] > 0.0f && isfinite(p.s[k]);
  }
  return p;
}

// Activity of every Gaussian (user order), the bounds of the active means and
// their number.  Reduced over the wave and the block first, and by a bounded
// number of blocks, since every global atomic here hits the same few words.
constexpr int kActiveBlocks = 1024;
__global__ __launch_bounds__(256) void k_active(int64_t n, const float *__restrict__ means,
                                                const float *__restrict__ log_scales,
                                                const float *__restrict__ quats,
                                                const float *__restrict__ density, float sigma_eps,
                                                uint8_t *__restrict__ active,
                                                uint32_t *__restrict__ bounds,
                                                int32_t *__restrict__ counters) {
  __shared__ uint32_t sb[kWavesPerBlock][6];
  __shared__ int32_t sc[kWavesPerBlock];
  uint32_t m[6] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0u, 0u, 0u};
  int32_t count = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const Params p = load_params(i, means, log_scales, quats, density, sigma_eps);
    active[i] = p.ok ? 1 : 0;
    if (p.ok) {
      count++;
      for (int k = 0; k < 3; k++) {
        const uint32_t u = f2ord(p.mu[k]);
        m[k] = min(m[k], u);
        m[3 + k] = max(m[3 + k], u);
      }
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    for (int k = 0; k < 3; k++) {
      m[k] = min(m[k], (uint32_t)__shfl_xor((int)m[k], o, 64));
      m[3 + k] = max(m[3 + k], (uint32_t)__shfl_xor((int)m[3 + k], o, 64));
    }
    count += __shfl_xor(count, o, 64);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) {
    for (int k = 0; k < 6; k++) sb[wid][k] = m[k];
    sc[wid] = count;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    uint32_t v = sb[0][threadIdx.x];
    for (int w = 1; w < kWavesPerBlock; w++)
      v = threadIdx.x < 3 ? min(v, sb[w][threadIdx.x]) : max(v, sb[w][threadIdx.x]);
    if (threadIdx.x < 3) atomicMin(&bounds[threadIdx.x], v);
    else atomicMax(&bounds[threadIdx.x], v);
  } else if (threadIdx.x == 6) {
    int32_t c = 0;
    for (int w = 0; w < kWavesPerBlock; w++) c += sc[w];
    if (c) atomicAdd(&counters[0], c);
  }
}

// The records of the active Gaussians, thread i the i-th in Z order: Sec. 3.1
// Eq. 1 and the sigma_eps level-set ellipsoid of Supp. B (geometry record,
// padded AABB), what the chain rule needs (aux), the collection's leaf test
// (sup) and the segment tree's leaf (empty past the active ones).  Computed in
// Z order straight from the parameters, 44 bytes gathered a Gaussian: as
// user-order records gathered afterwards it took 240 bytes more a Gaussian
// and four launches more.
__global__ __launch_bounds__(256) void k_records(int64_t P, const int32_t *__restrict__ counters,
                                                 const uint32_t *__restrict__ perm,
                                                 const float *__restrict__ means,
                                                 const float *__restrict__ log_scales,
                                                 const float *__restrict__ quats,
                                                 const float *__restrict__ density, float sigma_eps,
                                                 float4 *__restrict__ geom, float2 *__restrict__ aabb,
                                                 float4 *__restrict__ aux, float4 *__restrict__ sup,
                                                 float2 *__restrict__ seg) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  float2 *leaf = seg + 3 * (P + i);
  if (i >= counters[0]) {
    const float inf = __builtin_huge_valf();
    leaf[0] = make_float2(inf, inf);
    leaf[1] = make_float2(inf, -inf);
    leaf[2] = make_float2(-inf, -inf);
    return;
  }
  const Params p = load_params(perm[i], means, log_scales, quats, density, sigma_eps);
  const float *mu = p.mu, *s = p.s, *q = p.q;
  const float rn = rsqrtf(p.qn2), qn = sqrtf(p.qn2);
  const float w = q[0] * rn, x = q[1] * rn, y = q[2] * rn, z = q[3] * rn;
  float R[9];
  R[0] = 1.0f - 2.0f * (y * y + z * z); R[1] = 2.0f * (x * y - w * z); R[2] = 2.0f * (x * z + w * y);
  R[3] = 2.0f * (x * y + w * z); R[4] = 1.0f - 2.0f * (x * x + z * z); R[5] = 2.0f * (y * z - w * x);
  R[6] = 2.0f * (x * z - w * y); R[7] = 2.0f * (y * z + w * x); R[8] = 1.0f - 2.0f * (x * x + y * y);
  const float k2 = 2.0f * logf(p.sig / sigma_eps);
  const float k = sqrtf(k2);
  float M[9];
  // row r of M = S^-1 R^T is column r of R divided by s_r
  for (int r = 0; r < 3; r++)
    for (int c = 0; c < 3; c++) M[3 * r + c] = R[3 * c + r] / s[r];
  // minimal AABB half-lengths L_i = k sqrt(sum_j r_ij^2 s_j^2) (Supp. B), padded
  // outward so that every point of an FP32 ray/ellipsoid interval lies inside
  const float amax = fmaxf(fabsf(mu[0]), fmaxf(fabsf(mu[1]), fabsf(mu[2])));
  float lo[3], hi[3];
  for (int r = 0; r < 3; r++) {
    float acc = 0.0f;
    for (int c = 0; c < 3; c++) acc += R[3 * r + c] * R[3 * r + c] * s[c] * s[c];
    float L = k * sqrtf(acc);
    L = L * 1.0001f + 2e-6f * (amax + L) + 1e-30f;
    lo[r] = mu[r] - L;
    hi[r] = mu[r] + L;
  }
  // bounding sphere of the ellipsoid: radius k max(s), padded like L
  float rad = k * fmaxf(s[0], fmaxf(s[1], s[2]));
  rad = rad * 1.0001f + 2e-6f * (amax + rad) + 1e-30f;
  geom[4 * i] = make_float4(mu[0], mu[1], mu[2], k2);
  geom[4 * i + 1] = make_float4(M[0], M[1], M[2], M[3]);
  geom[4 * i + 2] = make_float4(M[4], M[5], M[6], M[7]);
  geom[4 * i + 3] = make_float4(M[8], p.sig, log2f(p.sig), 0.0f);
  aux[2 * i] = make_float4(s[0], s[1], s[2], q[0] / qn);
  aux[2 * i + 1] = make_float4(q[1] / qn, q[2] / qn, q[3] / qn, qn);
  // N = k S R^T
  const float k0 = k * s[0], k1 = k * s[1], k3 = k * s[2];
  sup[4 * i] = make_float4(mu[0], mu[1], mu[2], rad);
  sup[4 * i + 1] = make_float4(k0 * R[0], k0 * R[3], k0 * R[6], fmaxf(k0, fmaxf(k1, k3)));
  sup[4 * i + 2] = make_float4(k1 * R[1], k1 * R[4], k1 * R[7], 0.0f);
  sup[4 * i + 3] = make_float4(k3 * R[2], k3 * R[5], k3 * R[8], 0.0f);
  const float2 b0 = make_float2(lo[0], lo[1]), b1 = make_float2(lo[2], hi[0]),
               b2 = make_float2(hi[1], hi[2]);
  aabb[3 * i] = b0; aabb[3 * i + 1] = b1; aabb[3 * i + 2] = b2;
  leaf[0] = b0; leaf[1] = b1; leaf[2] = b2;
}

// Spherical-Gaussian lobes (user order): lobe j of the user record (amplitude
// rgb, axis xyz, sharpness) becomes (amplitude rgb, sharpness, unit axis,
// |xi|); absent lobes (j >= n_sg, a zero or non-finite axis) are all zero, so
// they add nothing to the colour and get no gradient.
__global__ __launch_bounds__(256) void k_sg_pack(int64_t n, int n_sg, const float *__restrict__ sg,
                                                 float *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  for (int j = 0; j < kMaxSg; j++) {
    float r[kSgLobeFloats] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (j < n_sg) {
      const float *p = sg + ((size_t)i * n_sg + j) * kSgUserFloats;
      const float xn = sqrtf(p[3] * p[3] + p[4] * p[4] + p[5] * p[5]);
      if (xn > 0.0f && isfinite(xn)) {
        r[0] = p[0]; r[1] = p[1]; r[2] = p[2];
        r[3] = p[6];
        r[4] = p[3] / xn; r[5] = p[4] / xn; r[6] = p[5] / xn;
        r[7] = xn;
      }
    }
    float4 *o = reinterpret_cast<float4 *>(out + (size_t)kSgFloats * i + kSgLobeFloats * j);
    o[0] = make_float4(r[0], r[1], r[2], r[3]);
    o[1] = make_float4(r[4], r[5], r[6], r[7]);
  }
}

// Spread the low 21 bits of v so that bit b lands at bit 3b.
__device__ __forceinline__ uint64_t spread3(uint64_t v) {
  v &= 0x1fffffull;
  v = (v | (v << 32)) & 0x1f00000000ffffull;
  v = (v | (v << 16)) & 0x1f0000ff0000ffull;
  v = (v | (v << 8)) & 0x100f00f00f00f00full;
  v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

// Z-order index of the normalised, quantised mean (Sec. 3.3).  Inactive
// Gaussians get the key 2^(3*bits), above every active key.
__device__ __forceinline__ uint64_t morton_key(int64_t i, const float *__restrict__ means,
                                               const uint8_t *__restrict__ active,
                                               const uint32_t *__restrict__ bounds, int bits) {
  if (!active[i]) return 1ull << (3 * bits);
  const float qmax = (float)((1u << bits) - 1u);
  uint64_t c[3];
  for (int k = 0; k < 3; k++) {
    const float lo = ord2f(bounds[k]), hi = ord2f(bounds[3 + k]);
    const float ext = hi - lo;
    float u = ext > 0.0f ? (means[3 * i + k] - lo) / ext : 0.0f;
    u = fminf(fmaxf(u, 0.0f), 1.0f);
    c[k] = (uint64_t)(u * qmax + 0.5f);
    if (c[k] > (uint64_t)qmax) c[k] = (uint64_t)qmax;
  }
  return (spread3(c[0]) << 2) | (spread3(c[1]) << 1) | spread3(c[2]);
}

__global__ __launch_bounds__(256) void k_morton(int64_t n, const float *__restrict__ means,
                                                const uint8_t *__restrict__ active,
                                                const uint32_t *__restrict__ bounds, int bits,
                                                uint64_t *__restrict__ keys,
                                                uint32_t *__restrict__ vals) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  keys[i] = morton_key(i, means, active, bounds, bits);
  vals[i] = (uint32_t)i;
}

// Up to kSmallSort Gaussians: keys and sort in one workgroup's LDS, a bitonic
// network over (key, index) -- the index makes the order that of a stable
// sort.  The passes below cost such a scene 25 launches of a few microseconds.
constexpr int kSmallSort = 4096;
__global__ __launch_bounds__(1024) void k_sort_small(int n, const float *__restrict__ means,
                                                     const uint8_t *__restrict__ active,
                                                     const uint32_t *__restrict__ bounds, int bits,
                                                     uint64_t *__restrict__ keys,
                                                     uint32_t *__restrict__ vals) {
  __shared__ uint64_t sk[kSmallSort];
  __shared__ uint32_t sv[kSmallSort];
  int p2 = 2;
  while (p2 < n) p2 <<= 1;
  for (int e = threadIdx.x; e < p2; e += 1024) {
    sk[e] = e < n ? morton_key(e, means, active, bounds, bits) : ~0ull;
    sv[e] = (uint32_t)e;
  }
  for (int k = 2; k <= p2; k <<= 1)
    for (int j = k >> 1; j >= 1; j >>= 1) {
      __syncthreads();
      for (int t = threadIdx.x; t < p2 / 2; t += 1024) {
        const int a = 2 * t - (t & (j - 1)), b = a + j;   // the t-th pair at distance j
        const uint64_t ka = sk[a], kb = sk[b];
        const uint32_t va = sv[a], vb = sv[b];
        const bool above = ka > kb || (ka == kb && va > vb);
        if (above == ((a & k) == 0)) {
          sk[a] = kb; sk[b] = ka;
          sv[a] = vb; sv[b] = va;
        }
      }
    }
  __syncthreads();
  for (int e = threadIdx.x; e < n; e += 1024) {
    keys[e] = sk[e];
    vals[e] = sv[e];
  }
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort, 8-bit digits.  Each block owns a tile of
// kSortItems keys; a pass is histogram -> exclusive scan of each digit's row
// over the blocks, one workgroup a digit -> stable scatter with per-wave
// ballot multisplit, every block adding up the 256 digit totals itself.  (One
// workgroup scanning all rows in turn took 56 of a pass's 83 us at 1M.)

constexpr int kSortThreads = 256;
constexpr int kSortRounds = 16;
constexpr int kSortItems = kSortThreads * kSortRounds;

__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint64_t *__restrict__ keys,
                                                             int64_t n, int shift,
                                                             uint32_t *__restrict__ hist,
                                                             int nblocks) {
  __shared__ uint32_t h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kSortItems;
  for (int r = 0; r < kSortRounds; r++) {
    const int64_t i = base + r * kSortThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 0xff], 1u);
  }
  __syncthreads();
  hist[(size_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// Inclusive scan of one value a thread over a 256-thread block.
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *wsum) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  __syncthreads();
  if (lane == 63) wsum[wid] = v;
  __syncthreads();
  for (int w = 0; w < wid; w++) v += wsum[w];
  return v;
}

// Row blockIdx.x (a digit) of the histogram: exclusive scan over the blocks in
// place, the row's total to totals[digit].
__global__ __launch_bounds__(kSortThreads) void k_scan_rows(uint32_t *__restrict__ hist, int nblocks,
                                                            uint32_t *__restrict__ totals) {
  __shared__ uint32_t wsum[kWavesPerBlock];
  __shared__ uint32_t last;
  uint32_t *row = hist + (size_t)blockIdx.x * nblocks;
  uint32_t carry = 0;
  for (int base = 0; base < nblocks; base += kSortThreads) {
    const int i = base + threadIdx.x;
    const uint32_t v = i < nblocks ? row[i] : 0u;
    const uint32_t x = block_scan(v, wsum);
    if (i < nblocks) row[i] = carry + x - v;
    if (threadIdx.x == kSortThreads - 1) last = x;
    __syncthreads();
    carry += last;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(
    const uint64_t *__restrict__ keys_in, const uint32_t *__restrict__ vals_in,
    uint64_t *__restrict__ keys_out, uint32_t *__restrict__ vals_out, int64_t n, int shift,
    const uint32_t *__restrict__ hist, int nblocks, const uint32_t *__restrict__ totals) {
  __shared__ uint32_t base[256];
  __shared__ uint32_t wcount[kWavesPerBlock][256];
  __shared__ uint32_t wsum[kWavesPerBlock];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t total = totals[threadIdx.x];
  base[threadIdx.x] = hist[(size_t)threadIdx.x * nblocks + blockIdx.x] + block_scan(total, wsum) - total;
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  const int64_t tile = (int64_t)blockIdx.x * kSortItems;
  for (int r = 0; r < kSortRounds; r++) {
    for (int w = 0; w < kWavesPerBlock; w++) wcount[w][threadIdx.x] = 0;
    __syncthreads();
    const int64_t i = tile + r * kSortThreads + threadIdx.x;
    const bool valid = i < n;
    uint64_t key = 0;
    uint32_t val = 0;
    uint32_t digit = 0;
    if (valid) { key = keys_in[i]; val = vals_in[i]; digit = (uint32_t)(key >> shift) & 0xffu; }
    // lanes of this wave holding the same digit
    uint64_t same = ballot(valid);
    for (int b = 0; b < 8; b++) {
      const uint64_t bal = ballot(((digit >> b) & 1u) != 0);
      same &= ((digit >> b) & 1u) ? bal : ~bal;
    }
    const uint32_t rank = (uint32_t)__popcll(same & lt_mask);
    if (valid && rank == 0) wcount[wid][digit] = (uint32_t)__popcll(same);
    __syncthreads();
    if (valid) {
      uint32_t off = base[digit] + rank;
      for (int w = 0; w < wid; w++) off += wcount[w][digit];
      keys_out[off] = key;
      vals_out[off] = val;
    }
    __syncthreads();
    uint32_t tot = 0;
    for (int w = 0; w < kWavesPerBlock; w++) tot += wcount[w][threadIdx.x];
    base[threadIdx.x] += tot;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Z-ordered pack: dst row i = src row perm[i].  One thread per destination
// float, so the reads of a source row are contiguous.
__global__ __launch_bounds__(256) void k_gather_rows(int64_t n, const int32_t *__restrict__ counters,
                                                     const uint32_t *__restrict__ perm,
                                                     const float *__restrict__ src, int src_stride,
                                                     int src_cols, float *__restrict__ dst,
                                                     int dst_stride) {
  const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = f / dst_stride;
  const int k = (int)(f - i * dst_stride);
  if (i >= n || i >= counters[0]) return;
  dst[f] = k < src_cols ? src[(size_t)perm[i] * src_stride + k] : 0.0f;
}

// Z-ordered colour records in the layout of the march's matrix operands:
// [channel][k][q] of coefficient m = 4q + k, zero past the degree, so that one
// 16-byte read gives a lane its coefficients of all four inner steps.  One
// thread per 16 bytes.
__global__ __launch_bounds__(256) void k_pack_colour(uint32_t n, const int32_t *__restrict__ counters,
                                                     const uint32_t *__restrict__ perm,
                                                     const float *__restrict__ sh, int sh_k,
                                                     float4 *__restrict__ col) {
  const uint32_t f = blockIdx.x * 256u + threadIdx.x;
  const uint32_t i = f / (kColFloats / 4), e = f - i * (kColFloats / 4);
  if (i >= n || (int)i >= counters[0]) return;
  const int ch = (int)e >> 2, k = (int)e & 3;
  const float *row = sh + (size_t)perm[i] * sh_k * 3 + ch;
  float v[4];
  for (int q = 0; q < 4; q++) v[q] = 4 * q + k < sh_k ? row[3 * (4 * q + k)] : 0.0f;
  col[f] = make_float4(v[0], v[1], v[2], v[3]);
}

// Node boxes without inter-thread synchronisation: a segment tree (heap
// layout, P leaves, P a power of two) over the Z-ordered leaf boxes gives the
// union of any leaf range in O(log P) reads; every internal node's child
// boxes are the unions of its two child ranges.
// Up to nine levels at once: a block takes 512 consecutive boxes of the level
// of `width` nodes to the one box above them.  (k_records writes the leaves.)
__device__ __forceinline__ void box_union(float *d, const float *a, const float *b) {
  for (int c = 0; c < 3; c++) { d[c] = fminf(a[c], b[c]); d[3 + c] = fmaxf(a[3 + c], b[3 + c]); }
}
__global__ __launch_bounds__(256) void k_seg_up(int64_t width, float *__restrict__ seg) {
  __shared__ float box[256 * 6];
  int64_t w = width >> 1;                      // nodes of the level written
  int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int m = (int)(w < 256 ? w : 256);            // of them in this block
  if ((int)threadIdx.x < m) {
    float a[12], d[6];
    const float4 *src = reinterpret_cast<const float4 *>(seg + 12 * (size_t)(w + k));
    for (int q = 0; q < 3; q++) {
      const float4 v = src[q];
      a[4 * q] = v.x; a[4 * q + 1] = v.y; a[4 * q + 2] = v.z; a[4 * q + 3] = v.w;
    }
    box_union(d, a, a + 6);
    for (int c = 0; c < 6; c++) seg[6 * (size_t)(w + k) + c] = box[6 * threadIdx.x + c] = d[c];
  }
  while (m > 1) {
    m >>= 1;
    w >>= 1;
    float d[6];
    __syncthreads();
    if ((int)threadIdx.x < m) box_union(d, box + 12 * threadIdx.x, box + 12 * threadIdx.x + 6);
    __syncthreads();
    if ((int)threadIdx.x < m) {
      k = (int64_t)blockIdx.x * m + threadIdx.x;
      for (int c = 0; c < 6; c++) seg[6 * (size_t)(w + k) + c] = box[6 * threadIdx.x + c] = d[c];
    }
  }
}

// Union of the boxes of leaves [l, r] (inclusive).
__device__ __forceinline__ void seg_query(const float *__restrict__ seg, int64_t P, int64_t l,
                                          int64_t r, float *box) {
  for (int c = 0; c < 3; c++) { box[c] = __builtin_huge_valf(); box[3 + c] = -__builtin_huge_valf(); }
  l += P;
  r += P + 1;
  while (l < r) {
    if (l & 1) {
      const float *x = seg + 6 * (size_t)l++;
      for (int c = 0; c < 3; c++) { box[c] = fminf(box[c], x[c]); box[3 + c] = fmaxf(box[3 + c], x[3 + c]); }
    }
    if (r & 1) {
      const float *x = seg + 6 * (size_t)(--r);
      for (int c = 0; c < 3; c++) { box[c] = fminf(box[c], x[c]); box[3 + c] = fmaxf(box[3 + c], x[3 + c]); }
    }
    l >>= 1;
    r >>= 1;
  }
}

// ---------------------------------------------------------------------------
// Karras LBVH over the sorted keys of the active Gaussians.  Internal node i
// covers a key range with i at one end; duplicate keys are split by index.
__device__ __forceinline__ int lcp(const uint64_t *__restrict__ k, int n, int i, int j) {
  if (j < 0 || j >= n) return -1;
  const uint64_t a = k[i], b = k[j];
  if (a == b) return 64 + __clz((uint32_t)(i ^ j));
  return __clzll(a ^ b);
}

__global__ __launch_bounds__(256) void k_lbvh_hierarchy(int64_t n_max,
                                                        const int32_t *__restrict__ counters,
                                                        const uint64_t *__restrict__ keys,
                                                        const float *__restrict__ aabb,
                                                        const float *__restrict__ seg, int64_t P,
                                                        float4 *__restrict__ nodes) {
  const int n = counters[0];
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (tid >= n_max) return;
  const int i = (int)tid;
  if (n == 1 && i == 0) {
    nodes[0] = make_float4(aabb[0], aabb[1], aabb[2], __int_as_float(~0));
    nodes[1] = make_float4(aabb[3], aabb[4], aabb[5], __int_as_float(kNoChild));
    nodes[2] = make_float4(0.f, 0.f, 0.f, __int_as_float(0));
    nodes[3] = make_float4(0.f, 0.f, 0.f, __int_as_float(0));
    return;
  }
  if (i >= n - 1) return;
  const int d = (lcp(keys, n, i, i + 1) - lcp(keys, n, i, i - 1)) >= 0 ? 1 : -1;
  const int dmin = lcp(keys, n, i, i - d);
  int64_t lmax = 2;
  while (lmax < 2 * (int64_t)n && lcp(keys, n, i, (int)(i + lmax * d)) > dmin) lmax <<= 1;
  int l = 0;
  for (int64_t t = lmax >> 1; t >= 1; t >>= 1) {
    const int64_t jj = i + (l + t) * d;
    if (jj >= 0 && jj < n && lcp(keys, n, i, (int)jj) > dmin) l += (int)t;
  }
  const int j = i + l * d;
  const int dnode = lcp(keys, n, i, j);
  int s = 0;
  int t = l;
  do {
    t = (t + 1) >> 1;
    if (lcp(keys, n, i, i + (s + t) * d) > dnode) s += t;
  } while (t > 1);
  const int gamma = i + s * d + (d < 0 ? -1 : 0);
  const int lo = i < j ? i : j, hi = i < j ? j : i;
  const int left = (lo == gamma) ? ~gamma : gamma;
  const int right = (hi == gamma + 1) ? ~(gamma + 1) : gamma + 1;
  float bl[6], br[6];
  seg_query(seg, P, lo, gamma, bl);
  seg_query(seg, P, gamma + 1, hi, br);
  float4 *nd = nodes + 4 * (size_t)i;
  nd[0] = make_float4(bl[0], bl[1], bl[2], __int_as_float(left));
  nd[1] = make_float4(bl[3], bl[4], bl[5], __int_as_float(right));
  // the node's leaf (Z index) range [lo, hi]; the split is implied by the
  // left link (gamma), so range-restricted traversals can prune children
  nd[2] = make_float4(br[0], br[1], br[2], __int_as_float(lo));
  nd[3] = make_float4(br[3], br[4], br[5], __int_as_float(hi));
}

// A 4-wide node by surface-area collapse: every binary internal node gathers
// its two children and then, while it has fewer than four, replaces the
// internal child of largest box surface area by that child's two children
// (in place, so the record stays in left-to-right Z order).  Every internal
// node gets a record, indexed by its binary index, so a link to an internal
// child is that child's binary index.
struct Node4 {
  int m;                 // children
  int lk[4], first[4], last[4];
  float4 lo[4], hi[4];
};
__device__ __forceinline__ Node4 collapse4(int i, int n_inner, const float4 *__restrict__ nodes) {
  int lk[4];
  float4 blo[4], bhi[4];
  int m = 0;
  {
    const float4 a = nodes[4 * (size_t)i], b = nodes[4 * (size_t)i + 1], c = nodes[4 * (size_t)i + 2],
                 d = nodes[4 * (size_t)i + 3];
    const int l0 = __float_as_int(a.w), l1 = __float_as_int(b.w);
    if (l0 != kNoChild) { lk[m] = l0; blo[m] = a; bhi[m] = b; m++; }
    if (l1 != kNoChild) { lk[m] = l1; blo[m] = c; bhi[m] = d; m++; }
  }
  while (m < 4) {
    int best = -1;
    float bsa = -1.0f;
    for (int k = 0; k < m; k++) {
      if (lk[k] < 0 || lk[k] >= n_inner) continue;
      const float dx = bhi[k].x - blo[k].x, dy = bhi[k].y - blo[k].y, dz = bhi[k].z - blo[k].z;
      const float sa = dx * dy + dy * dz + dz * dx;
      if (sa > bsa) { bsa = sa; best = k; }
    }
    if (best < 0) break;
    const int x = lk[best];
    const float4 a = nodes[4 * (size_t)x], b = nodes[4 * (size_t)x + 1], c = nodes[4 * (size_t)x + 2],
                 d = nodes[4 * (size_t)x + 3];
    const int l0 = __float_as_int(a.w), l1 = __float_as_int(b.w);
    if (l0 == kNoChild || l1 == kNoChild) break;   // only the root of a one-leaf tree has one child
    for (int k = m; k > best + 1; k--) { lk[k] = lk[k - 1]; blo[k] = blo[k - 1]; bhi[k] = bhi[k - 1]; }
    lk[best] = l0; blo[best] = a; bhi[best] = b;
    lk[best + 1] = l1; blo[best + 1] = c; bhi[best + 1] = d;
    m++;
  }
  Node4 r;
  r.m = m;
  for (int k = 0; k < 4; k++) {
    r.lk[k] = kNoChild;
    r.first[k] = 1;      // empty range
    r.last[k] = 0;
    r.lo[k] = r.hi[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (k >= m) continue;
    r.lk[k] = lk[k];
    r.lo[k] = blo[k];
    r.hi[k] = bhi[k];
    r.first[k] = r.last[k] = ~lk[k];
    if (lk[k] >= 0) {
      r.first[k] = __float_as_int(nodes[4 * (size_t)lk[k] + 2].w);
      r.last[k] = __float_as_int(nodes[4 * (size_t)lk[k] + 3].w);
    }
  }
  return r;
}

// The marching kernels' form, 128 bytes (kQuadFloats).
__global__ __launch_bounds__(256) void k_quads(int64_t n_max, const int32_t *__restrict__ counters,
                                               const float4 *__restrict__ nodes,
                                               float4 *__restrict__ quads) {
  const int n = counters[0];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int n_inner = n > 1 ? n - 1 : 1;
  if (i >= n_max || n <= 0 || i >= n_inner) return;
  const Node4 r = collapse4((int)i, n_inner, nodes);
  float4 *qd = quads + (size_t)(kQuadFloats / 4) * i;
  for (int k = 0; k < 4; k++) {
    const float lo[3] = {r.lo[k].x, r.lo[k].y, r.lo[k].z}, hi[3] = {r.hi[k].x, r.hi[k].y, r.hi[k].z};
    float c[3] = {0.0f, 0.0f, 0.0f}, h[3] = {0.0f, 0.0f, 0.0f};
    if (k < r.m)
      for (int a = 0; a < 3; a++) {
        // half-extents rounded outward: [c - h, c + h] holds [lo, hi]
        c[a] = 0.5f * lo[a] + 0.5f * hi[a];
        h[a] = fmaf(fabsf(c[a]), 4e-7f, fmaxf(hi[a] - c[a], c[a] - lo[a]) * 1.000002f);
      }
    qd[2 * k] = make_float4(c[0], c[1], c[2], h[0]);
    qd[2 * k + 1] = make_float4(h[1], h[2], __int_as_float(r.lk[k]),
                                __int_as_float(k < r.m ? r.first[k] : 0x7fffffff));
  }
}

// The debug call's form, 144 bytes: plain boxes, links and leaf ranges.
__global__ __launch_bounds__(256) void k_nodes4(int64_t n_max, const int32_t *__restrict__ counters,
                                                const float4 *__restrict__ nodes,
                                                float *__restrict__ nodes4) {
  const int n = counters[0];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int n_inner = n > 1 ? n - 1 : 1;
  if (i >= n_max || n <= 0 || i >= n_inner) return;
  const Node4 r = collapse4((int)i, n_inner, nodes);
  float *f = nodes4 + (size_t)kNode4Floats * i;
  for (int k = 0; k < 4; k++) {
    f[6 * k] = r.lo[k].x; f[6 * k + 1] = r.lo[k].y; f[6 * k + 2] = r.lo[k].z;
    f[6 * k + 3] = r.hi[k].x; f[6 * k + 4] = r.hi[k].y; f[6 * k + 5] = r.hi[k].z;
    f[24 + k] = __int_as_float(r.lk[k]);
    f[28 + 2 * k] = __int_as_float(r.first[k]);
    f[29 + 2 * k] = __int_as_float(r.last[k]);
  }
}

// ---------------------------------------------------------------------------
static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

hipError_t launch_build(const BuildArgs &a, hipStream_t st) {
  const int64_t n = a.n;
  k_build_init<<<1, 64, 0, st>>>(a.bounds, a.counters);
  k_active<<<std::min(nblk(n, 256), (unsigned)kActiveBlocks), 256, 0, st>>>(
      n, a.means, a.log_scales, a.quats, a.density, a.sigma_eps, a.active, a.bounds, a.counters);
  int cur = 0;
  if (n <= kSmallSort) {
    k_sort_small<<<1, 1024, 0, st>>>((int)n, a.means, a.active, a.bounds, a.morton_bits, a.keys[0],
                                     a.vals[0]);
  } else {
    k_morton<<<nblk(n, 256), 256, 0, st>>>(n, a.means, a.active, a.bounds, a.morton_bits, a.keys[0],
                                           a.vals[0]);
    const int nb = (int)nblk(n, kSortItems);
    const int passes = (3 * a.morton_bits + 1 + 7) / 8;
    uint32_t *totals = a.sort_hist + (size_t)256 * nb;
    for (int p = 0; p < passes; p++) {
      const int shift = 8 * p;
      k_radix_hist<<<nb, kSortThreads, 0, st>>>(a.keys[cur], n, shift, a.sort_hist, nb);
      k_scan_rows<<<256, kSortThreads, 0, st>>>(a.sort_hist, nb, totals);
      k_radix_scatter<<<nb, kSortThreads, 0, st>>>(a.keys[cur], a.vals[cur], a.keys[cur ^ 1],
                                                   a.vals[cur ^ 1], n, shift, a.sort_hist, nb, totals);
      cur ^= 1;
    }
  }
  *a.sorted_sel = cur;
  const uint32_t *perm = a.vals[cur];
  int64_t P = 1;
  while (P < n) P <<= 1;
  k_records<<<nblk(P, 256), 256, 0, st>>>(
      P, a.counters, perm, a.means, a.log_scales, a.quats, a.density, a.sigma_eps,
      reinterpret_cast<float4 *>(a.geom), reinterpret_cast<float2 *>(a.aabb),
      reinterpret_cast<float4 *>(a.aux), reinterpret_cast<float4 *>(a.sup),
      reinterpret_cast<float2 *>(a.seg));
  k_pack_colour<<<nblk(n * (kColFloats / 4), 256), 256, 0, st>>>(
      (uint32_t)n, a.counters, perm, a.sh, a.sh_k, reinterpret_cast<float4 *>(a.col));
  if (a.n_sg > 0) {
    k_sg_pack<<<nblk(n, 256), 256, 0, st>>>(n, a.n_sg, a.sg, a.sg_user);
    k_gather_rows<<<nblk(n * kSgFloats, 256), 256, 0, st>>>(n, a.counters, perm, a.sg_user,
                                                           kSgFloats, kSgFloats, a.sgrec, kSgFloats);
  }
  for (int64_t w = P; w > 1; w = w > 512 ? w >> 9 : 1)
    k_seg_up<<<nblk(w, 512), 256, 0, st>>>(w, a.seg);
  k_lbvh_hierarchy<<<nblk(n, 256), 256, 0, st>>>(n, a.counters, a.keys[cur], a.aabb, a.seg, P,
                                                 reinterpret_cast<float4 *>(a.nodes));
  k_quads<<<nblk(n, 256), 256, 0, st>>>(n, a.counters, reinterpret_cast<const float4 *>(a.nodes),
                                        reinterpret_cast<float4 *>(a.quads));
  return hipGetLastError();
}

hipError_t launch_nodes4(int64_t n, const int32_t *counters, const float *nodes, float *nodes4,
                         hipStream_t st) {
  k_nodes4<<<nblk(n, 256), 256, 0, st>>>(n, counters, reinterpret_cast<const float4 *>(nodes), nodes4);
  return hipGetLastError();
}

}  // namespace rgx
