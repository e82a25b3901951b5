// Forward and backward ray marching through the Gaussian field (Sec. 3.1
// Eq. 1-3; Sec. 3.2 Algorithm 1, Eq. 4-5).
//
// Execution model: one wave64 (one workgroup) owns one tile of 64 rays, or in
// small calls of 32 or 16, each shared by 2 or 4 lanes that take its samples
// between them.  Each lane marches its ray segment by segment (Alg. 1).  Candidate Gaussians come
// from a per-wave window list: for a depth window covering one or more
// segments of every live lane, a node-parallel walk of the LBVH gathers the
// Gaussians that may meet the packet of rays in its windows, each with
// conservative depth bounds (see trav_run).  Every segment then runs over
// that list with a wave-uniform depth pre-check, so one BVH walk serves
// several segments and its memory latency is spread over 64 independent node
// fetches per round.  A window too large for the list is processed in Z-index
// chunks: the walk pauses when the list is full and resumes after the chunk.
// The geometry of 64 list entries is fetched at once, one entry per lane; each
// group of four candidates takes its ray directions from the matrix cores and
// the rest with readlane (for_each_candidate).  The forward reads colour
// records at wave-uniform addresses through the scalar cache.  Closest-hit restarts
// beyond the window use a depth-first packet traversal, nearer child first.
//
// Every ray meets its Gaussians in Z-index order (window lists and their
// chunks are sorted, brute force counts up), whatever packet, window, tile
// shape or ray order is used; the images of all these variants are
// therefore bit-identical.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"
#include "tiles.hpp"


namespace rgx {

constexpr float kInf = __builtin_huge_valf();
constexpr float kHalfLog2e = 0.72134752044448170f;  // log2(e) / 2

struct Ray {
  float ox, oy, oz;  // wave-uniform camera centre
  float dx, dy, dz;  // unit direction
  float ix, iy, iz;  // 1 / direction (components clamped away from 0)
};

__device__ __forceinline__ float safe_inv(float d) {
  const float a = fabsf(d) < 1e-20f ? copysignf(1e-20f, d) : d;
  return 1.0f / a;
}

// Slab test of a (padded) AABB over the lane's interval [lo, hi], with the
// box's parametric range widened by a few ulps (robust traversal).
__device__ __forceinline__ bool box_hit(float lx, float ly, float lz, float hx, float hy, float hz,
                                        const Ray &r, float lo, float hi) {
  const float tx0 = (lx - r.ox) * r.ix, tx1 = (hx - r.ox) * r.ix;
  const float ty0 = (ly - r.oy) * r.iy, ty1 = (hy - r.oy) * r.iy;
  const float tz0 = (lz - r.oz) * r.iz, tz1 = (hz - r.oz) * r.iz;
  float bmin = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fminf(tz0, tz1));
  float bmax = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fmaxf(tz0, tz1));
  bmin = fmaf(-fabsf(bmin), 1e-6f, bmin);
  bmax = fmaf(fabsf(bmax), 1e-6f, bmax);
  return fmaxf(bmin, lo) <= fminf(bmax, hi);
}

// Entry parameter over [lo, hi] of a box of the 4-wide nodes (centre,
// half-extents), widened by 1e-6 of the distances involved, or +inf when the
// box misses the interval.
__device__ __forceinline__ float ray_box_entry(const vf4 &q0, const vf4 &q1, const Ray &r, float lo,
                                               float hi) {
  const float tx = (q0.x - r.ox) * r.ix, ty = (q0.y - r.oy) * r.iy, tz = (q0.z - r.oz) * r.iz;
  const float ex = fmaf(fabsf(tx), 1e-6f, q0.w * fabsf(r.ix)),
              ey = fmaf(fabsf(ty), 1e-6f, q1.x * fabsf(r.iy)),
              ez = fmaf(fabsf(tz), 1e-6f, q1.y * fabsf(r.iz));
  const float e = fmaxf(fmaxf(tx - ex, ty - ey), fmaxf(tz - ez, lo));
  return e <= fminf(fminf(tx + ex, ty + ey), fminf(tz + ez, hi)) ? e : kInf;
}

// Geometry of one Gaussian (wave-uniform, from the scalar cache).
struct Gauss {
  float mx, my, mz, k2;
  float m[9];
  float sig, l2sig;
  float ox, oy, oz;        // the camera centre in the local frame, M (o - mu) (with_origin)
};

// Fills the local-frame camera centre (shared by every ray of a wave).
__device__ __forceinline__ Gauss with_origin(Gauss g, float ox, float oy, float oz) {
  const float ex = ox - g.mx, ey = oy - g.my, ez = oz - g.mz;
  g.ox = fmaf(g.m[0], ex, fmaf(g.m[1], ey, g.m[2] * ez));
  g.oy = fmaf(g.m[3], ex, fmaf(g.m[4], ey, g.m[5] * ez));
  g.oz = fmaf(g.m[6], ex, fmaf(g.m[7], ey, g.m[8] * ez));
  return g;
}

__device__ __forceinline__ Gauss load_gauss(const float *geom, int j) {
  cfloat4p p = as_const4(geom) + 4 * j;
  const vf4 a = p[0], b = p[1], c = p[2], d = p[3];
  Gauss g;
  g.mx = a.x; g.my = a.y; g.mz = a.z; g.k2 = a.w;
  g.m[0] = b.x; g.m[1] = b.y; g.m[2] = b.z; g.m[3] = b.w;
  g.m[4] = c.x; g.m[5] = c.y; g.m[6] = c.z; g.m[7] = c.w;
  g.m[8] = d.x; g.sig = d.y; g.l2sig = d.z;
  return g;
}

// Ray / ellipsoid {q <= k^2}: q(t) = A (t - t*)^2 + h^2 about the point of
// closest approach; the chord is t* -/+ sqrt((k^2 - h^2) / A).
struct Chord {
  float A, ts, h2, tin, tout;
  bool exists;   // (chord_local, chord)
};

// The ray in the Gaussian's local frame (g carries the origin, with_origin).
__device__ __forceinline__ void ray_local(const Gauss &g, const Ray &r, float &opx, float &opy,
                                          float &opz, float &dpx, float &dpy, float &dpz) {
  opx = g.ox;
  opy = g.oy;
  opz = g.oz;
  dpx = fmaf(g.m[0], r.dx, fmaf(g.m[1], r.dy, g.m[2] * r.dz));
  dpy = fmaf(g.m[3], r.dx, fmaf(g.m[4], r.dy, g.m[5] * r.dz));
  dpz = fmaf(g.m[6], r.dx, fmaf(g.m[7], r.dy, g.m[8] * r.dz));
}

// From the ray's local-frame origin (opx, opy, opz) and direction.
__device__ __forceinline__ Chord chord_local(float opx, float opy, float opz, float dpx, float dpy,
                                             float dpz, float k2) {
  Chord c;
  c.A = fmaf(dpx, dpx, fmaf(dpy, dpy, dpz * dpz));
  const float B = fmaf(opx, dpx, fmaf(opy, dpy, opz * dpz));
  const float rA = __builtin_amdgcn_rcpf(c.A);
  c.ts = -B * rA;
  const float px = fmaf(c.ts, dpx, opx), py = fmaf(c.ts, dpy, opy), pz = fmaf(c.ts, dpz, opz);
  c.h2 = fmaf(px, px, fmaf(py, py, pz * pz));
  c.exists = c.h2 <= k2;
  const float w = __builtin_amdgcn_sqrtf(fmaxf(k2 - c.h2, 0.0f) * rA);
  c.tin = c.ts - w;
  c.tout = c.ts + w;
  return c;
}

__device__ __forceinline__ Chord chord(const Gauss &g, const Ray &r) {
  float opx, opy, opz, dpx, dpy, dpz;
  ray_local(g, r, opx, opy, opz, dpx, dpy, dpz);
  return chord_local(opx, opy, opz, dpx, dpy, dpz, g.k2);
}

// Colour of a Gaussian at the lane's direction: c = sum_m f_m Y_m.  Every
// colour record is kColFloats long whatever the degree (zero past sh_k) and
// Y_m = 0 for m >= sh_k, so the record is read at fixed offsets, without
// branches, and the terms past the degree add exact zeros.  The record's
// three 64-byte scalar loads (colour_load) can be issued ahead of work that
// does not need them, so that their latency overlaps it (colour_eval).
struct ColRec {
  vf4 f[kColFloats / 4];
};

__device__ __forceinline__ ColRec colour_load(const float *col, int j) {
  cfloat4p p = as_const4(col) + (size_t)(kColFloats / 4) * j;
  ColRec c;
#pragma unroll
  for (int q = 0; q < kColFloats / 4; q++) c.f[q] = p[q];
  // a scheduling barrier: the compiler would otherwise place the loads
  // just before their first use, and their latency would not overlap the
  // caller's work between colour_load and colour_eval
  __builtin_amdgcn_sched_barrier(0);
  return c;
}

__device__ __forceinline__ void colour_eval(const ColRec &rc, const float *Y, float &cr, float &cg,
                                            float &cb) {
  float acc[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int m = 0; m < 16; m++)
#pragma unroll
    for (int c = 0; c < 3; c++)   // coefficient m = 4q + k of channel c: [c][k][q]
      acc[c] = fmaf(rc.f[4 * c + (m & 3)][m >> 2], Y[m], acc[c]);
  cr = acc[0]; cg = acc[1]; cb = acc[2];
}

// Spherical-Gaussian lobes of Gaussian j added to the lane's colour:
// c += a_k exp(lambda_k (u_k.d - 1)) for the kMaxSg packed lobes (absent
// lobes have a = 0).  One lobe (two 16-byte scalar loads) per iteration, so
// the lobes do not all hold scalar registers at once.
__device__ __forceinline__ void sg_colour(const float *sg, int j, float dx, float dy, float dz,
                                          float &cr, float &cg, float &cb) {
  cfloat4p p = as_const4(sg) + (size_t)(kSgFloats / 4) * j;
#pragma unroll 1
  for (int k = 0; k < kMaxSg; k++) {
    const vf4 a = p[2 * k], u = p[2 * k + 1];
    const float cosang = fmaf(u.x, dx, fmaf(u.y, dy, u.z * dz));
    const float g = __builtin_amdgcn_exp2f(a.w * kLog2e * (cosang - 1.0f));
    cr = fmaf(a.x, g, cr);
    cg = fmaf(a.y, g, cg);
    cb = fmaf(a.z, g, cb);
  }
}

// Wave-uniform DFS stack, entry i held by lane i % 64 of s0 .. s4.  The
// closest-hit walk pushes at most 3 entries per 4-wide record on its current
// path (the record's unvisited children).  The records sit at binary internal
// nodes, each strictly deeper than the one before it on a path, and binary
// internal nodes lie at most 86 levels deep (the Karras split positions grow
// strictly down the tree over the 63-bit key extended by a 23-bit index), so
// a path meets at most 87 records and the stack never holds more than 261
// entries: 320 always suffice.
struct WaveStack {
  int s0 = 0, s1 = 0, s2 = 0, s3 = 0, s4 = 0, sp = 0, lane = 0;
  __device__ __forceinline__ bool push(int v) {
    if (sp < 64) s0 = lane == sp ? v : s0;
    else if (sp < 128) s1 = lane == sp - 64 ? v : s1;
    else if (sp < 192) s2 = lane == sp - 128 ? v : s2;
    else if (sp < 256) s3 = lane == sp - 192 ? v : s3;
    else if (sp < 320) s4 = lane == sp - 256 ? v : s4;
    else return false;
    sp++;
    return true;
  }
  __device__ __forceinline__ int pop() {
    sp--;
    const int q = sp >> 6, l = sp & 63;
    return q == 0 ? __builtin_amdgcn_readlane(s0, l)
         : q == 1 ? __builtin_amdgcn_readlane(s1, l)
         : q == 2 ? __builtin_amdgcn_readlane(s2, l)
         : q == 3 ? __builtin_amdgcn_readlane(s3, l)
                  : __builtin_amdgcn_readlane(s4, l);
  }
};

// Ends the compiler's freedom to sink a load towards its first use: the
// value must be in registers here, so loads written together are issued
// together and waited for once (empty asm statements, no instruction).
// pin_loaded: a per-lane (vector) value; pin_uniform: a wave-uniform one
// from the scalar cache.
__device__ __forceinline__ void pin_loaded(const vf4 &x) {
  asm volatile("" : : "v"(x.x), "v"(x.y), "v"(x.z), "v"(x.w));
}
__device__ __forceinline__ void pin_uniform(float x) { asm volatile("" : : "s"(x)); }
__device__ __forceinline__ void pin_lane(uint32_t x) { asm volatile("" : : "v"(x)); }

// ---------------------------------------------------------------------------
// Work distribution: global tile index -> view, pixel, output ray.

struct Pixel {
  int view, px, py, ray;
  bool valid;
};

// `lane` is the ray's number in its tile of `rays` rays.
__device__ __forceinline__ Pixel tile_pixel(const ViewTable &vt, const MarchOpts &op, int w,
                                            int lane, int rays) {
  int v = 0;
  while (v + 1 < vt.n_views && vt.v[v + 1].tile_begin <= w) v++;
  const View &V = vt.v[v];
  const int t = w - V.tile_begin;
  Pixel p;
  p.view = v;
  if (op.ray_order == 0) {
    const int r = t * rays + lane;
    p.valid = r < V.width * V.height;
    p.px = r % V.width;
    p.py = r / V.width;
  } else {
    int tx, ty;
    if (V.tile_order) {
      const uint32_t code = V.tile_order[t];
      tx = tile_column(code);
      ty = tile_row(code);
    } else {
      ty = t / V.tiles_x;
      tx = t - ty * V.tiles_x;
    }
    p.px = tx * op.tile_w + (lane & (op.tile_w - 1));
    p.py = ty * op.tile_h + (lane >> op.tile_w_log2);
    p.valid = p.px < V.width && p.py < V.height;
  }
  p.ray = V.ray_begin + p.py * V.width + p.px;
  return p;
}

// Whether this launch marches the view (the same answer in every wave, and in
// the backward of the same structure build).
__device__ __forceinline__ bool marches_view(const SceneDev &s, const MarchOpts &op, const View &V) {
  if (op.views == VIEWS_ALL) return true;
  bool inside = true;
#pragma unroll
  for (int k = 0; k < 3; k++)
    inside = inside && V.c2w[4 * k + 3] >= ord2f(s.bounds[k]) && V.c2w[4 * k + 3] <= ord2f(s.bounds[3 + k]);
  return uniform_int(inside ? 1 : 0) == (op.views == VIEWS_INSIDE ? 1 : 0);
}

__device__ __forceinline__ bool marches_any(const SceneDev &s, const MarchOpts &op, const ViewTable &vt) {
  if (op.views == VIEWS_ALL) return true;
  for (int v = 0; v < vt.n_views; v++)
    if (marches_view(s, op, vt.v[v])) return true;
  return false;
}

// A wave-uniform value held in a vector register: the camera centre is read
// throughout the march, and scalar registers are the scarcer resource there.
__device__ __forceinline__ float in_vgpr(float x) {
  float y;
  asm volatile("v_mov_b32 %0, %1" : "=v"(y) : "s"(x));
  return y;
}

__device__ __forceinline__ Ray make_ray(const View &V, int px, int py) {
  Ray r;
  r.ox = in_vgpr(V.c2w[3]); r.oy = in_vgpr(V.c2w[7]); r.oz = in_vgpr(V.c2w[11]);
  const float u = ((float)px + 0.5f - V.cx) / V.fx;
  const float v = ((float)py + 0.5f - V.cy) / V.fy;
  float dx = fmaf(V.c2w[0], u, fmaf(V.c2w[1], v, V.c2w[2]));
  float dy = fmaf(V.c2w[4], u, fmaf(V.c2w[5], v, V.c2w[6]));
  float dz = fmaf(V.c2w[8], u, fmaf(V.c2w[9], v, V.c2w[10]));
  const float inv = rsqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
  r.dx = dx * inv; r.dy = dy * inv; r.dz = dz * inv;
  r.ix = safe_inv(r.dx); r.iy = safe_inv(r.dy); r.iz = safe_inv(r.dz);
  return r;
}

// Non-persistent launches: block b -> a contiguous run of tiles per XCD
// (blocks are dealt to the 8 XCDs round robin).
__device__ __forceinline__ int xcd_block(int b, int nb) {
  const int q = nb >> 3, rem = nb & 7, x = b & 7, rank = b >> 3;
  return x * q + min(x, rem) + rank;
}

// Persistent launches: 8 queues, one contiguous chunk of tiles each; a wave
// drains its home queue, then the others.  Returns -1 when all are empty.
__device__ __forceinline__ int pop_tile(int32_t *queue, int n_tiles, int home, int lane) {
  const int per = (n_tiles + 7) >> 3;
  for (int k = 0; k < 8; k++) {
    const int qi = (home + k) & 7;
    const int begin = qi * per;
    const int len = min(per, n_tiles - begin);
    if (len <= 0) continue;
    int got = 0;
    if (lane == 0) got = atomicAdd(&queue[qi], 1);
    got = uniform_int(got);
    if (got < len) return begin + got;
  }
  return -1;
}

// Midpoint sample positions of a segment, t_k = o + (i0 + k + 1/2) dt: on the
// fixed grid o = t_n and i0 = N_s * segment index, otherwise o = a, i0 = 0.
// Held as t_0 and dt, t_k = t_0 + k dt (two registers instead of N_s).
struct Samples {
  float t0, dt;
  __device__ __forceinline__ float t(int k) const { return fmaf((float)k, dt, t0); }
};

// Eq. 5 with d_i = a (unit direction from the camera centre).
__device__ __forceinline__ float adaptive_dt(const MarchOpts &op, float a, float T) {
  const float base = fmaxf(a * op.inv_beta, op.dt_min);
  const float v = base * __builtin_amdgcn_exp2f(-__builtin_amdgcn_logf(T) * (1.0f / 3.0f));
  return v < op.dt_max ? v : op.dt_max;
}

// Per-lane segment state shared by forward and backward.
struct SegState {
  bool alive, pending;
  int seg_i;
  float a, cl_lo;
};


// The sample weights of one Gaussian for one lane:
// w_k = sigma~ exp(-q(t_k)/2) if q(t_k) <= k^2 else 0.  With t_k = t_0 + k dt
// and q(t) = A (t - t*)^2 + h^2, the exponent log2 sigma~ - q_k log2(e)/2 is
// a quadratic in the sample index, e_0 + k e_1 + k^2 e_2, so each sample
// costs two FMAs before its exp2; the truncation test q_k <= k^2 is the
// same quadratic against log2 sigma~ - k^2 log2(e)/2.
struct SampleExp {
  float e0, e1, e2, e_min;
  __device__ __forceinline__ float at(int k) const {
    return k == 0 ? e0 : fmaf((float)(k * k), e2, fmaf((float)k, e1, e0));
  }
  // a per-lane sample index (the same value at the same index)
  __device__ __forceinline__ float at(float k) const { return fmaf(k * k, e2, fmaf(k, e1, e0)); }
};

__device__ __forceinline__ SampleExp sample_exp(float k2, float l2sig, const Chord &c,
                                                const Samples &sp) {
  const float u0 = sp.t0 - c.ts;
  const float Au0 = c.A * u0;
  SampleExp x;
  x.e0 = fmaf(-fmaf(Au0, u0, c.h2), kHalfLog2e, l2sig);
  x.e1 = -kHalfLog2e * (2.0f * Au0 * sp.dt);
  x.e2 = -kHalfLog2e * (c.A * sp.dt * sp.dt);
  x.e_min = fmaf(-k2, kHalfLog2e, l2sig);
  return x;
}

// Segment bounds [a, b], step and sample positions of a live lane.
template <int NS>
__device__ __forceinline__ bool segment(const MarchOpts &op, bool grid, const SegState &ss,
                                        float tn, float T, float &a, float &b, float &dt,
                                        Samples &sp) {
  a = grid ? fmaf((float)(ss.seg_i * NS), op.dt, tn) : ss.a;
  dt = op.adaptive ? adaptive_dt(op, a, T) : op.dt;
  b = grid ? fmaf((float)((ss.seg_i + 1) * NS), op.dt, tn) : fmaf((float)NS, dt, a);
  sp.t0 = grid ? fmaf((float)(ss.seg_i * NS) + 0.5f, dt, tn) : fmaf(0.5f, dt, a);
  sp.dt = dt;
  return b > a;
}

// Restart at a closest hit t: on the fixed grid the segment holding t (never
// going back), otherwise t itself.
__device__ __forceinline__ void restart_at(const MarchOpts &op, float tn, float dS, float t,
                                           SegState &ss) {
  if (!op.adaptive && op.ess == 1) ss.seg_i = max(ss.seg_i, (int)floorf((t - tn) / dS));
  else ss.a = t;
}

// Next segment after [a, b]: the following one, or after an empty segment
// with skipping on, the closest hit `best` (kInf: unknown here -> query).
__device__ __forceinline__ void step_after(const MarchOpts &op, bool grid, bool nonempty, float best,
                                           float tn, float dS, float b, SegState &ss) {
  if (grid) ss.seg_i += 1;
  else ss.a = b;
  if (nonempty || !op.ess) return;
  if (best < kInf) restart_at(op, tn, dS, best, ss);
  else { ss.pending = true; ss.cl_lo = b; }
}

// Cross-lane helpers (gfx950): v_permlane32_swap / v_permlane16_swap exchange
// halves / rows between two registers; DPP row and quad permutes.
__device__ __forceinline__ float swap32_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                  false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
typedef float f4v __attribute__((ext_vector_type(4)));

// 4x4 transposition between four registers and the wave's four 16-lane rows:
// row q of x[g] becomes row g of x[q].
__device__ __forceinline__ void transpose_rows(float (&x)[4]) {
  uint32_t u[4];
#pragma unroll
  for (int g = 0; g < 4; g++) u[g] = __float_as_uint(x[g]);
#pragma unroll
  for (int g = 0; g < 2; g++) {
    const auto p = __builtin_amdgcn_permlane32_swap(u[g], u[g + 2], false, false);
    u[g] = p[0];
    u[g + 2] = p[1];
  }
#pragma unroll
  for (int g = 0; g < 4; g += 2) {
    const auto p = __builtin_amdgcn_permlane16_swap(u[g], u[g + 1], false, false);
    u[g] = p[0];
    u[g + 1] = p[1];
  }
#pragma unroll
  for (int g = 0; g < 4; g++) x[g] = __uint_as_float(u[g]);
}
// A tile of 64 / S rays: the lanes ray, ray + 64 / S, ... hold one ray, each
// some of its samples.  out[i] is the value of the ray's lane i, in all of
// its lanes.
template <int S>
__device__ __forceinline__ void ray_lanes(float x, float (&out)[S]) {
  if constexpr (S == 1) {
    out[0] = x;
  } else {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    if constexpr (S == 2) {
      out[0] = __uint_as_float(p[0]);
      out[1] = __uint_as_float(p[1]);
    } else {
      const auto a = __builtin_amdgcn_permlane16_swap(p[0], p[0], false, false);
      const auto b = __builtin_amdgcn_permlane16_swap(p[1], p[1], false, false);
      out[0] = __uint_as_float(a[0]);
      out[1] = __uint_as_float(a[1]);
      out[2] = __uint_as_float(b[0]);
      out[3] = __uint_as_float(b[1]);
    }
  }
}
__device__ __forceinline__ float uniform_lane(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
// In-row DPP permute of x; a lane with no valid source keeps `id`.
template <int CTRL>
__device__ __forceinline__ float dpp_or(float x, float id) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(id), __float_as_int(x), CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
// Minimum over the wave of values that are never negative (+inf allowed;
// -0 counts as 0), without LDS traffic: the bit patterns of such floats
// order as signed integers, so each in-row DPP permute (quad xor 1, quad
// xor 2, half-row mirror, row mirror) is one fused integer minimum, leaving
// each row's minimum in every lane of the row; the four rows are then read
// back.
__device__ __forceinline__ float wave_min_nonneg_dpp(float v) {
  int x = __float_as_int(v);
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0xb1, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x4e, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x141, 0xf, 0xf, false));
  x = min(x, __builtin_amdgcn_update_dpp(0x7fffffff, x, 0x140, 0xf, 0xf, false));
  const int a = min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16));
  const int b = min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48));
  return __int_as_float(min(a, b));
}


// One reduce-scatter stage over DPP partners: of 2H values per lane, the
// half picked by lane bit BIT is kept and the partner's other half added (the
// partner must differ from the lane in that bit).
template <int H, int CTRL, int BIT>
__device__ __forceinline__ void dpp_stage_bit(float *x, int lane) {
  const bool up = (lane & BIT) != 0;
#pragma unroll
  for (int i = 0; i < H; i++) {
    const float keep = up ? x[i + H] : x[i];
    const float send = up ? x[i] : x[i + H];
    x[i] = keep + dpp<CTRL>(send);
  }
}

// Sum over the wave of 16 per-lane slots.  Two half-wave swaps halve the
// slots per lane (lane bits 5 and 4 pick the half kept), two in-row DPP
// stages halve them again (bits 3 and 2, with the row and half-row mirrors
// as partners), and a quad sum completes the total.  Lane L returns the wave
// total of slot (L >> 2) & 15.
__device__ __forceinline__ float wave_sum_slots16(const float *g, int lane) {
  float y[8], z[4];
#pragma unroll
  for (int i = 0; i < 8; i++) y[i] = swap32_sum(g[i], g[i + 8]);
#pragma unroll
  for (int i = 0; i < 4; i++) z[i] = swap16_sum(y[i], y[i + 4]);
  dpp_stage_bit<2, 0x140, 8>(z, lane);   // row_mirror: lane p <-> 15 - p
  dpp_stage_bit<1, 0x141, 4>(z, lane);   // row_half_mirror: p <-> 7 - p within 8
  float u = z[0];
  u += dpp<0xb1>(u);                     // quad_perm [1,0,3,2]
  u += dpp<0x4e>(u);                     // quad_perm [2,3,0,1]
  return u;
}

// SH-coefficient gradients of a batch of up to 16 Gaussians, a small dense
// product on the matrix cores.  For Gaussian b of the batch and channel c,
// dL/df_{m,c} = sum over the tile's rays r of Y_m(d_r) G_c(r) S_b(r), S_b(r)
// the ray's sum over samples of w_k T_k phi_k (zero where the ray misses b).
// With A_c[m][r] = Y_m(d_r) G_c(r) (Y held in registers, G in LDS)
// and B[r][b] = S_b(r) staged in LDS, each channel is 16 chained 16x16x4 FP32
// MFMAs over the 64 rays, computed transposed: D_c = B^T A_c^T, so that the
// result holds Gaussians in rows and coefficients in columns.  Operand
// layout of v_mfma_f32_16x16x4_f32 (wave64): first operand X[i][k] in lane
// i + 16k, second Y[k][j] in lane j + 16k, D[i][j] in lane j + 16 (i / 4),
// register i % 4.  Each atomic instruction therefore adds 16 consecutive
// floats (one 64-byte line) to each of 4 Gaussians' rows.
constexpr int kSbStride = 66;   // floats per staged row: transposed reads hit distinct banks

constexpr int kRowStride = 17;   // floats per lane of the transposition: distinct banks both ways

// Sums of 16 slots over the 16 lanes of each row: lane L returns slot L & 15
// summed over row L >> 4.  Through LDS, 16 writes and 16 reads that cost the
// vector units 15 additions: in registers (two half-wave swaps, two in-row
// stages, a quad sum) a Gaussian's 16 slots took 12 row swaps of 8 cycles and
// 23 other instructions, 76 ns of a full SIMD against about 20.
__device__ __forceinline__ float sum_rows16(float *buf, const float *v, int lane) {
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int e = 0; e < 16; e++) buf[lane * kRowStride + e] = v[e];
  __builtin_amdgcn_wave_barrier();
  const float *p = buf + (lane & 48) * kRowStride + (lane & 15);
  float x[16];
#pragma unroll
  for (int i = 0; i < 16; i++) x[i] = p[i * kRowStride];
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int h = 8; h >= 1; h >>= 1)
#pragma unroll
    for (int i = 0; i < h; i++) x[i] += x[i + h];
  return x[0];
}

struct ShBatch {
  float y[16];      // Y_m of rays 4q + (lane >> 4), row m = lane & 15
  int n = 0;        // uniform: staged Gaussians
  int id = 0;       // lane b < 16: the Gaussian staged in row b
};

// LDS of the batch: the staged S rows and the tile's G, channel by channel.
// A_c is formed from Y and G at every product (one multiplication beside
// three matrix instructions): held whole it took 32 more registers, and the
// kernel spilled.
template <bool ROWS>
struct ShMem {
  float s[16 * kSbStride];
  float g[3][64];
  float r[ROWS ? 64 * kRowStride : 1];   // a Gaussian's slots, lane by lane (sum_rows16)
};

// Y and G of a new tile.
template <bool ROWS>
__device__ __forceinline__ void sh_batch_start(ShBatch &B, ShMem<ROWS> &sm, const float *Y, float g0,
                                               float g1, float g2, int lane) {
#pragma unroll
  for (int m = 0; m < 16; m++) sm.s[m * kSbStride + lane] = Y[m];
  sm.g[0][lane] = g0;
  sm.g[1][lane] = g1;
  sm.g[2][lane] = g2;
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int q = 0; q < 16; q++) B.y[q] = sm.s[(lane & 15) * kSbStride + 4 * q + (lane >> 4)];
  __builtin_amdgcn_wave_barrier();
  B.n = 0;
}

// Multiplies out the staged batch and adds it to the accumulators.
template <bool ROWS>
__device__ __forceinline__ void sh_batch_flush(ShBatch &B, const ShMem<ROWS> &sm, float *acc, int sh_k,
                                               int lane) {
  if (B.n == 0) return;
  __builtin_amdgcn_wave_barrier();
  f4v d0 = {0.0f, 0.0f, 0.0f, 0.0f}, d1 = d0, d2 = d0;
#pragma unroll
  for (int q = 0; q < 16; q++) {
    // S_b(r) for Gaussian b = lane & 15 and ray r = 4q + (lane >> 4)
    const int ray = 4 * q + (lane >> 4);
    const float sv = sm.s[(lane & 15) * kSbStride + ray];
    d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(sv, B.y[q] * sm.g[0][ray], d0, 0, 0, 0);
    d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(sv, B.y[q] * sm.g[1][ray], d1, 0, 0, 0);
    d2 = __builtin_amdgcn_mfma_f32_16x16x4f32(sv, B.y[q] * sm.g[2][ray], d2, 0, 0, 0);
  }
  // lane: coefficient m = lane & 15 of Gaussians 4 (lane >> 4) + i
  const int m = lane & 15;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int b = 4 * (lane >> 4) + i;
    const int jb = __shfl(B.id, b, 64);
    if (b < B.n && m < sh_k) {
      float *row = acc + (size_t)kAccFloats * jb + 16;
      unsafeAtomicAdd(row + m, d0[i]);
      unsafeAtomicAdd(row + 16 + m, d1[i]);
      unsafeAtomicAdd(row + 32 + m, d2[i]);
    }
  }
  __builtin_amdgcn_wave_barrier();
  B.n = 0;
}

__device__ __forceinline__ float wave_sum_f(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return uniform_float(v);
}
// Wave minimum and maximum (exact, so the order of the reduction does not
// matter) without LDS traffic: four in-row DPP permutes (quad xor 1, quad
// xor 2, half-row mirror, row mirror) leave each row's extreme in every lane
// of the row, and the four rows are read out.  Called with the whole wave
// active.
__device__ __forceinline__ float wave_min(float v) {
  v = fminf(v, dpp_or<0xb1>(v, kInf));
  v = fminf(v, dpp_or<0x4e>(v, kInf));
  v = fminf(v, dpp_or<0x141>(v, kInf));
  v = fminf(v, dpp_or<0x140>(v, kInf));
  const float a = fminf(uniform_lane(v, 0), uniform_lane(v, 16));
  const float b = fminf(uniform_lane(v, 32), uniform_lane(v, 48));
  return fminf(a, b);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_or<0xb1>(v, -kInf));
  v = fmaxf(v, dpp_or<0x4e>(v, -kInf));
  v = fmaxf(v, dpp_or<0x141>(v, -kInf));
  v = fmaxf(v, dpp_or<0x140>(v, -kInf));
  const float a = fmaxf(uniform_lane(v, 0), uniform_lane(v, 16));
  const float b = fmaxf(uniform_lane(v, 32), uniform_lane(v, 48));
  return fmaxf(a, b);
}

// Closest hit (Alg. 1 ClosestHit, Eq. 4) for the lanes with `pending` set:
// min over Gaussians whose chord meets [cl_lo, t_far] of max(t_in, cl_lo).
// Depth-first packet traversal, nearer child first (by the smallest entry
// over the wave's pending lanes); each lane's bound shrinks to its best hit
// so far and prunes.  A minimum does not depend on the visiting order.
// Query qn of ray `ray`: recorded into (or, for q < kReplayK, replayed from)
// op.replay when op.replay_mode asks for it.
template <int S>
__device__ __forceinline__ void closest_pass(const SceneDev &s, const MarchOpts &op, int n_active,
                                             const Ray &r, float tn, float tf, float dS,
                                             SegState &ss, int32_t *err, int32_t *st_closest,
                                             int &qn, int64_t ray) {
  if (ballot(ss.pending) == 0) return;
  const int st_lane = __lane_id();
  const bool replayed = op.replay_mode == 2 && ss.pending && qn < kReplayK;
  const float rbest = replayed ? op.replay[ray * kReplayK + qn] : kInf;
  const bool search = ss.pending && !replayed;
  const float lo = search ? ss.cl_lo : kInf;
  float hi = search ? tf : -kInf;
  float best = kInf;
  // Every candidate value max(t_in, lo) is at least lo: a lane whose best
  // reached lo has its answer and leaves the search (hi below lo), so that
  // the boxes around a ray starting inside ellipsoids are not all walked.
  auto leaf = [&](int j) {
    const Gauss g = with_origin(load_gauss(s.geom, j), r.ox, r.oy, r.oz);
    const Chord c = chord(g, r);
    if (c.exists && c.tin <= hi && c.tout >= lo) {
      best = fminf(best, fmaxf(c.tin, lo));
      hi = best <= lo ? -kInf : fminf(hi, best);
    }
  };
  __builtin_amdgcn_s_setprio(3);   // a dependent walk, as the collection's
  if (ballot(search) == 0) {
    // every pending lane replays
  } else if (op.brute_force) {
    for (int j = 0; j < n_active; j++) leaf(j);
  } else if (n_active > 0) {
    const int n_inner = n_active > 1 ? n_active - 1 : 1;
    WaveStack st;
    st.lane = st_lane;
    st.sp = 0;
    int node = 0, visits = 0;
    for (;;) {
      if (ballot(hi >= lo) == 0) break;   // every searching lane has its answer
      if (node < 0) {
        if (st.sp == 0) break;
        const int v = st.pop();
        if (v < 0) { leaf(~v); continue; }
        node = v;
      }
      if (++visits > n_inner) { if (err) *err = 2; break; }
      int link[4];
      float e[4];
      if constexpr (S > 1) {
        // the lanes of a ray take the four children between them
        const int child = st_lane / (64 / S);
        const vf4 *np = reinterpret_cast<const vf4 *>(s.quads) + (kQuadFloats / 4) * (size_t)node;
        vf4 q0[4 / S], q1[4 / S];
#pragma unroll
        for (int t = 0; t < 4 / S; t++) {
          q0[t] = np[2 * (child + S * t)];
          q1[t] = np[2 * (child + S * t) + 1];
        }
#pragma unroll
        for (int t = 0; t < 4 / S; t++) {
          float x = ray_box_entry(q0[t], q1[t], r, lo, hi);
          x = fminf(x, dpp_or<0xb1>(x, kInf));
          x = fminf(x, dpp_or<0x4e>(x, kInf));
          x = fminf(x, dpp_or<0x141>(x, kInf));
          x = fminf(x, dpp_or<0x140>(x, kInf));
#pragma unroll
          for (int c = 0; c < S; c++) {
            constexpr int kR = 64 / S;
            const int ch = c + S * t;
            link[ch] = __builtin_amdgcn_readlane(__float_as_int(q1[t].z), kR * c);
            e[ch] = uniform_lane(x, kR * c);
            if constexpr (S == 2) e[ch] = fminf(e[ch], uniform_lane(x, kR * c + 16));
            if (link[ch] == kNoChild) e[ch] = kInf;
          }
        }
      } else {
        cfloat4p np = as_const4(s.quads) + (kQuadFloats / 4) * (size_t)node;
        vf4 q[kQuadFloats / 4];
#pragma unroll
        for (int k = 0; k < kQuadFloats / 4; k++) q[k] = np[k];
        // the boxes and links go out as one batch of loads: the box tests and
        // the link checks below would otherwise each wait for a load of their
        // own
#pragma unroll
        for (int k = 0; k < kQuadFloats / 4; k++) { pin_uniform(q[k].x); pin_uniform(q[k].z); }
#pragma unroll
        for (int k = 0; k < 4; k++) {
          link[k] = __float_as_int(q[2 * k + 1].z);
          e[k] = link[k] != kNoChild
                     ? wave_min_nonneg_dpp(ray_box_entry(q[2 * k], q[2 * k + 1], r, lo, hi))
                     : kInf;
        }
      }
      // links out of range (a malformed tree) end the walk; checked after
      // the box tests, which do not need them, in one branch-free test
      int bad = 0;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const int lk = link[k];
        bad |= (lk != kNoChild) & (lk >= 0 ? lk >= n_inner : ~lk >= n_active);
      }
      if (bad) { if (err) *err = 3; break; }
      // nearest child next; the others on the stack, farthest first (the
      // entries are wave-uniform, so this small sort is uniform too)
#pragma unroll
      for (int x = 0; x < 3; x++)
#pragma unroll
        for (int y = 0; y < 3 - x; y++)
          if (e[y + 1] < e[y]) {
            const float te = e[y]; e[y] = e[y + 1]; e[y + 1] = te;
            const int tl = link[y]; link[y] = link[y + 1]; link[y + 1] = tl;
          }
      bool overflow = false;
#pragma unroll
      for (int k = 3; k >= 1; k--)
        if (e[k] < kInf && !st.push(link[k])) overflow = true;
      if (overflow) { if (err) *err = 1; break; }
      if (!(e[0] < kInf)) { node = -1; continue; }
      if (link[0] >= 0) node = link[0];
      else { leaf(~link[0]); node = -1; }
    }
  }
  __builtin_amdgcn_s_setprio(0);
  if (ss.pending) {
    if (replayed) best = rbest;
    else if (op.replay_mode == 1 && qn < kReplayK && st_lane < 64 / S) op.replay[ray * kReplayK + qn] = best;
    qn++;
    if (st_closest) (*st_closest)++;
    if (!(best < kInf)) ss.alive = false;
    else restart_at(op, tn, dS, best, ss);
    ss.pending = false;
  }
}

// ---------------------------------------------------------------------------
// Window collection.  For a per-lane depth window [lo, hi] the wave gathers
// every Gaussian that may meet some lane's window, restricted to the Z-index
// range [z0, z1), with a conservative depth interval for each.  Every test is
// against the packet as a whole: the bounding cone of the rays (apex at the
// shared camera centre) and the shell between the nearest window start and
// the farthest window end, applied to the boxes of 4-wide nodes and to the
// leaves' ellipsoids.  Exact per-ray chords are left to the segment loop,
// which computes them anyway.  The traversal is node-parallel: the frontier of
// (node, first leaf) is an LDS stack ordered by first leaf, smallest on top;
// each round takes the (up to) 64 lowest subtrees, four lanes to a node and
// one child box to a lane, and their children go back on top in order -- a
// 64-wide depth-first walk in Z order, whose frontier stays narrow.  What
// bounds it is memory latency and the cache's rate of scattered 16-byte reads:
// a quad reads its node's 128 bytes as whole lines (two reads a lane for four
// children, against four 64-byte gathers for two children of a binary node),
// and a round of 64 nodes does the work of three binary ones.  1M Gaussians,
// 4 x 1024x768: 13.1k binary nodes a tile -> 6.7k, forward 39.7 -> 34.5 ms;
// 1920x1080 frame 21.0 -> 17.7 ms; 5M Gaussians, 257x193: 95 -> 75 ms.
// When
// the frontier or the list would overflow, z1 is lowered (a radix select over
// the pending Z indices) and everything at or beyond it is dropped, so the
// result is always complete for [z0, z1); the caller continues from z1 with
// another chunk.  The list is finally sorted by Z index, so every ray meets
// its Gaussians in Z order whatever window, chunking or packet produced the
// list -- the order of brute force.

constexpr int kRingCap = 256;    // frontier (stack) entries
constexpr int kStageCap = 320;   // staged leaves; a round adds at most 4 per node
constexpr int kListCap = 512;    // window list entries (multiple of 64, at most 512)

struct ListMem {
  uint16_t order[kListCap];        // slots of the current chunk's entries, in Z-index order
  int32_t l_id[kListCap];
  float l_tin[kListCap], l_tout[kListCap];
  int32_t cand[64];                // a block's candidates, packed to the front
};

struct WaveMem : ListMem {
  float rlo[64], rhi[64];          // the rays' windows
  struct {                         // traversal state, kept while a collection is paused
    int2 ring[kRingCap];           // (4-wide node, its first leaf)
    int32_t st_id[kStageCap];
  } c;
};

// Statistics only: the tile's rays and their AABB-only leaf counts.
struct StatMem {
  float rdx[64], rdy[64], rdz[64], rix[64], riy[64], riz[64];
  int32_t cnt_box[64];
};
template <bool STATS> struct StatMemOf {};
template <> struct StatMemOf<true> : StatMem {};

__device__ __forceinline__ uint64_t join64(uint32_t lo, uint32_t hi) {
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Set bits of a mask in the lanes before this one.
__device__ __forceinline__ int count_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

__device__ __forceinline__ uint64_t lanes_below(int lane) {
  return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Lane-local ray r from the wave's LDS copy (origin is wave-uniform).
__device__ __forceinline__ Ray lds_ray(const StatMem &M, const Ray &self, int r) {
  Ray q;
  q.ox = self.ox; q.oy = self.oy; q.oz = self.oz;
  q.dx = M.rdx[r]; q.dy = M.rdy[r]; q.dz = M.rdz[r];
  q.ix = M.rix[r]; q.iy = M.riy[r]; q.iz = M.riz[r];
  return q;
}

// Loads one geometry record at a per-lane address (vector memory path).
__device__ __forceinline__ Gauss load_gauss_lane(const float *geom, int j) {
  const vf4 *p = reinterpret_cast<const vf4 *>(geom) + 4 * j;
  const vf4 a = p[0], b = p[1], c = p[2], d = p[3];
  Gauss g;
  g.mx = a.x; g.my = a.y; g.mz = a.z; g.k2 = a.w;
  g.m[0] = b.x; g.m[1] = b.y; g.m[2] = b.z; g.m[3] = b.w;
  g.m[4] = c.x; g.m[5] = c.y; g.m[6] = c.z; g.m[7] = c.w;
  g.m[8] = d.x; g.sig = d.y; g.l2sig = d.z;
  return g;
}

// Largest z in [zlo, zhi] such that at most `target` of the wave's values
// (V per lane, where ok) are below z.  zlo, zhi and the result are uniform.
template <int V>
__device__ __forceinline__ int select_cut(const int (&v)[V], const bool (&ok)[V], int zlo, int zhi,
                                          int target) {
  while (zlo < zhi) {
    const int mid = zlo + ((zhi - zlo + 1) >> 1);
    int c = 0;
#pragma unroll
    for (int k = 0; k < V; k++) c += __popcll(ballot(ok[k] && v[k] < mid));
    if (c <= target) zlo = mid;
    else zhi = mid - 1;
  }
  return zlo;
}

// Keeps the list entries with index < z1 (order preserved); returns the
// count.  64 entries at a time: a write never passes an unread entry.
__device__ __forceinline__ int compact_list(WaveMem &M, int lane, int count, int z1) {
  const uint64_t below = lanes_below(lane);
  int base = 0;
  for (int e0 = 0; e0 < count; e0 += 64) {
    const int e = e0 + lane;
    int id = 0;
    float tin = 0.0f, tout = 0.0f;
    bool keep = false;
    if (e < count) {
      id = M.l_id[e];
      tin = M.l_tin[e];
      tout = M.l_tout[e];
      keep = id < z1;
    }
    __builtin_amdgcn_wave_barrier();
    const uint64_t b = ballot(keep);
    if (keep) {
      const int pos = base + __popcll(b & below);
      M.l_id[pos] = id;
      M.l_tin[pos] = tin;
      M.l_tout[pos] = tout;
    }
    base += __popcll(b);
    __builtin_amdgcn_wave_barrier();
  }
  return base;
}

// Keeps the frontier entries in [head, tail) whose first leaf is below z1
// (order preserved, same scheme); returns the new end.
__device__ __forceinline__ int compact_ring(WaveMem &M, int lane, int head, int tail, int z1) {
  const uint64_t below = lanes_below(lane);
  int base = head;
  for (int e0 = head; e0 < tail; e0 += 64) {
    const int e = e0 + lane;
    int2 v = make_int2(0, 0);
    bool keep = false;
    if (e < tail) {
      v = M.c.ring[e];
      keep = v.y < z1;
    }
    __builtin_amdgcn_wave_barrier();
    const uint64_t b = ballot(keep);
    if (keep) {
      M.c.ring[base + __popcll(b & below)] = v;
    }
    base += __popcll(b);
    __builtin_amdgcn_wave_barrier();
  }
  return base;
}

// In-lane stage of the register bitonic sort: element 64q + lane is paired
// with 64(q ^ JQ) + lane (the same lane).
template <int JQ>
__device__ __forceinline__ void bitonic_inlane(uint32_t (&key)[8], int k, int nq) {
#pragma unroll
  for (int q = 0; q < 8; q++) {
    const int p = q ^ JQ;
    if (p > q && p < nq) {
      const bool up = ((64 * q) & k) == 0;
      const uint32_t x = key[q], y = key[p];
      const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
      key[q] = up ? lo : hi;
      key[p] = up ? hi : lo;
    }
  }
}

// Orders the list entries with index below zc by Gaussian (Z) index (the
// other entries stay in the list for a later chunk): the keys (index << 9 |
// slot; indices are distinct and below 2^23) are sorted by a bitonic network
// held in registers, element 64q + lane in key[q] -- partners in other lanes
// are read with cross-lane shuffles, partners in the same lane are registers.
// The sorted slots go to M.order.  Returns how many there are.
__device__ __forceinline__ int sort_list(WaveMem &M, int lane, int count, int zc) {
  static_assert(kListCap <= 512, "sort keys hold a 9-bit slot");
  int p2 = 64;
  while (p2 < count) p2 <<= 1;
  const int nq = p2 >> 6;
  uint32_t key[8];
  int valid = 0;
#pragma unroll
  for (int q = 0; q < 8; q++) {
    const int e = 64 * q + lane;
    const int id = e < count ? M.l_id[e] : 0x7fffffff;
    key[q] = id < zc ? ((uint32_t)id << 9) | (uint32_t)e : 0xffffffffu;
    valid += __popcll(ballot(id < zc));
  }
  for (int k = 2; k <= p2; k <<= 1) {
    for (int j = k >> 1; j >= 1; j >>= 1) {
      if (j >= 64) {
        if (j == 64) bitonic_inlane<1>(key, k, nq);
        else if (j == 128) bitonic_inlane<2>(key, k, nq);
        else bitonic_inlane<4>(key, k, nq);
      } else {
        const bool lower = (lane & j) == 0;
#pragma unroll
        for (int q = 0; q < 8; q++) {
          if (q < nq) {
            const uint32_t x = key[q];
            const uint32_t y = (uint32_t)__shfl_xor((int)x, j, 64);
            const bool up = ((64 * q + lane) & k) == 0;
            const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
            key[q] = up == lower ? lo : hi;
          }
        }
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int q = 0; q < 8; q++) {
    const int e = 64 * q + lane;
    if (e < valid) M.order[e] = (uint16_t)(key[q] & 511u);
  }
  __builtin_amdgcn_wave_barrier();
  return valid;
}

// The packet bound: apex o, unit axis u, half-angle (cos, sin) padded
// outward, and the depth shell [t_lo, t_hi] (distances from o).  Rays spread
// too far for the angular tests leave `narrow` false and get (cos, sin) =
// (0, 1), with which the box test only keeps the half-space ahead.
struct Cone {
  float ux, uy, uz, cs, sn, t_lo, t_hi;
  float du;      // bound of |d - u| over the rays
  bool narrow;
};

__device__ __forceinline__ Cone packet_cone(const WaveMem &M, const Ray &self, int lane,
                                            uint64_t rays) {
  const bool mine = (rays >> lane) & 1;
  const float sx = wave_sum_f(mine ? self.dx : 0.0f), sy = wave_sum_f(mine ? self.dy : 0.0f),
              sz = wave_sum_f(mine ? self.dz : 0.0f);
  Cone k;
  const float n2 = fmaf(sx, sx, fmaf(sy, sy, sz * sz));
  const float inv = n2 > 0.0f ? rsqrtf(n2) : 0.0f;
  k.ux = sx * inv; k.uy = sy * inv; k.uz = sz * inv;
  // sine and cosine of each ray's angle to the axis (cross product: no
  // cancellation at small angles)
  const float cx = self.dy * k.uz - self.dz * k.uy, cy = self.dz * k.ux - self.dx * k.uz,
              cz = self.dx * k.uy - self.dy * k.ux;
  const float sn = wave_max(mine ? sqrtf(fmaf(cx, cx, fmaf(cy, cy, cz * cz))) : 0.0f);
  const float cs = wave_min(mine ? fmaf(self.dx, k.ux, fmaf(self.dy, k.uy, self.dz * k.uz)) : 1.0f);
  k.narrow = n2 > 0.0f && cs > 0.5f;
  k.sn = fminf(sn * 1.0001f + 2e-6f, 1.0f);
  k.cs = sqrtf(fmaxf(1.0f - k.sn * k.sn, 0.0f));
  if (!k.narrow) { k.sn = 1.0f; k.cs = 0.0f; }
  k.du = k.sn * sqrtf(2.0f / (1.0f + k.cs));
  k.t_lo = wave_min(mine ? M.rlo[lane] : kInf);
  k.t_hi = wave_max(mine ? M.rhi[lane] : -kInf);
  return k;
}

// Conservative test of a box (centre v relative to the apex, half-extents h)
// against the packet: false only if no point of the box lies on a ray of the
// packet at a depth inside the shell.  The box's exact distance from the apex
// bounds the depth from below (near the apex, inside dense clusters, an axial
// bound is weaker: 1.2M Gaussians of an outdoor scene, 1600x1063, 19.1k leaf
// tests a tile against 17.8k and 29.7 ms against 28.3 ms).
// From above, along the axis the box reaches v.u + h.|u|, and a ray point at
// depth t lies in [t cos, t].
// Across it, with p = v - (v.u) u, every box point has a distance of at least
// |p| - h.|p| / |p| from the axis, and a cone point at most tan times its
// axial coordinate; the inequality is taken times |p| to need no division.
// Margins: 2e-5 of the distance (rounding of v, v.u and p), 1e-3 of the
// box's extent across.  Every comparison rejects, so that the NaN of a box with
// infinite sides (a Gaussian whose squared scale overflows, and every node
// above it) keeps it.
__device__ __forceinline__ bool cone_box(const Cone &k, float vx, float vy, float vz, float hx,
                                         float hy, float hz) {
  const float al = fmaf(vx, k.ux, fmaf(vy, k.uy, vz * k.uz));
  const float ru = fmaf(hx, fabsf(k.ux), fmaf(hy, fabsf(k.uy), hz * fabsf(k.uz)));
  const float px = fmaf(-al, k.ux, vx), py = fmaf(-al, k.uy, vy), pz = fmaf(-al, k.uz, vz);
  const float p2 = fmaf(px, px, fmaf(py, py, pz * pz));
  const float rp = fmaf(hx, fabsf(px), fmaf(hy, fabsf(py), hz * fabsf(pz)));
  const float pw = __builtin_amdgcn_sqrtf(p2);
  const float pad = fmaf(fabsf(al) + pw, 2e-5f, 1e-6f);
  const float far = al + ru + pad;
  const float qx = fmaxf(fabsf(vx) - hx, 0.0f), qy = fmaxf(fabsf(vy) - hy, 0.0f),
              qz = fmaxf(fabsf(vz) - hz, 0.0f);
  const float near2 = fmaf(qx, qx, fmaf(qy, qy, qz * qz)), reach = k.t_hi + pad;
  return !(near2 > reach * reach) & !(far < k.t_lo * k.cs) & !(far < 0.0f) &
         !(fmaf(-1.001f, rp, p2) * k.cs > fmaf(far, k.sn, pad) * pw);
}

// Depth bounds of the packet's rays inside a sphere (centre v relative to the
// apex, radius rho), and whether the sphere can meet the packet at all; used
// for packets too wide for the ellipsoid's own test.
__device__ __forceinline__ bool cone_sphere(const Cone &k, float vx, float vy, float vz, float rho,
                                            float *dlo, float *dhi) {
  const float d = sqrtf(fmaf(vx, vx, fmaf(vy, vy, vz * vz)));
  // rho's margin covers the FP32 chord ends near tangency (~3e-4 of the extent)
  const float pad = fmaf(d, 1e-5f, rho * 1.001f);
  *dlo = d - pad;
  *dhi = d + pad;
  const float al = fmaf(vx, k.ux, fmaf(vy, k.uy, vz * k.uz));
  return !(*dlo > k.t_hi) & !(*dhi < k.t_lo) & !(al + pad < 0.0f);
}

// Depth bounds [lo, hi] of every ray of a narrow packet inside one ellipsoid,
// and whether the ellipsoid can meet the packet at all (returned).  v is its
// centre relative to the apex, N = k S R^T (rows n0..n2), so that |N x| is its
// support along a unit x, and kmax = k max(s).  A point o + t d of it
// satisfies |t - v.d| <= |N d|; v.d ranges over [|v| cos(phi + theta),
// |v| cos(phi - theta)] for the angle phi between v and the axis, and
// |N d| <= |N u| + kmax |d - u|.  The cone: every point p of the ellipsoid has
// |p_perp| >= perp - r_w and p.u <= al + r_u, r_w = |N p| / perp and r_u =
// |N u| its supports along the unit perpendicular of the centre and along the
// axis (the inequality taken times perp).
__device__ __forceinline__ bool cone_ellipsoid(const Cone &k, float vx, float vy, float vz,
                                               const vf4 &n0, const vf4 &n1, const vf4 &n2,
                                               float kmax, float rad, float *lo, float *hi) {
  const float w0 = fmaf(n0.x, k.ux, fmaf(n0.y, k.uy, n0.z * k.uz));
  const float w1 = fmaf(n1.x, k.ux, fmaf(n1.y, k.uy, n1.z * k.uz));
  const float w2 = fmaf(n2.x, k.ux, fmaf(n2.y, k.uy, n2.z * k.uz));
  const float ru = __builtin_amdgcn_sqrtf(fmaf(w0, w0, fmaf(w1, w1, w2 * w2)));
  const float ext = fmaf(kmax, k.du, ru);
  const float d = __builtin_amdgcn_sqrtf(fmaf(vx, vx, fmaf(vy, vy, vz * vz)));
  const float al = fmaf(vx, k.ux, fmaf(vy, k.uy, vz * k.uz));
  const float px = fmaf(-al, k.ux, vx), py = fmaf(-al, k.uy, vy), pz = fmaf(-al, k.uz, vz);
  const float p2 = fmaf(px, px, fmaf(py, py, pz * pz));
  const float perp = __builtin_amdgcn_sqrtf(p2);
  // phi >= theta <=> perp cos(theta) >= al sin(theta); phi <= 90 deg <=> al >= 0
  const float c_hi = perp * k.cs >= al * k.sn ? fmaf(al, k.cs, perp * k.sn) : d;
  const float c_lo = al >= 0.0f ? fmaf(al, k.cs, -perp * k.sn) : -d;
  // margins: FP32 chord ends near tangency, rounding of N and the norms
  const float pad = fmaf(ext, 1e-3f, fmaf(d, 2e-5f, 1e-6f));
  // (the bounding sphere's own depth range is the tighter one off the axis)
  const float out = fmaf(rad, 1e-3f, rad + pad);
  *lo = fmaxf(c_lo - ext - pad, d - out);
  *hi = fminf(c_hi + ext + pad, d + out);
  const float y0 = fmaf(n0.x, px, fmaf(n0.y, py, n0.z * pz));
  const float y1 = fmaf(n1.x, px, fmaf(n1.y, py, n1.z * pz));
  const float y2 = fmaf(n2.x, px, fmaf(n2.y, py, n2.z * pz));
  const float rwp = __builtin_amdgcn_sqrtf(fmaf(y0, y0, fmaf(y1, y1, y2 * y2)));
  // (rejecting comparisons, as in cone_box)
  return !(*lo > k.t_hi) & !(*hi < k.t_lo) &
         !(fmaf(-1.001f, rwp, p2) * k.cs > fmaf(al + ru, k.sn, pad) * perp);
}

// Wave-uniform state of a window collection.  The list holds the entries
// found so far; the frontier stack and the staged leaves live in M.c.  A
// collection ends either complete for [z0, z1) (z1 may have been lowered by a
// cut) or paused: the list is full, and its entries below zp -- everything
// below the smallest pending Z index -- form a complete chunk [z0, zp); after
// that chunk, trav_advance drops those entries and trav_run resumes.
struct Trav {
  uint64_t rays;                   // lanes whose windows (M.rlo, M.rhi) are collected
  int z0, z1, zp;
  int sp, staged, count, visits;
  bool paused;
};

__device__ __forceinline__ void trav_start(WaveMem &M, int lane, Trav &t, uint64_t rays, int z0,
                                           int z1) {
  t.rays = rays;
  t.z0 = z0;
  t.z1 = z1;
  t.zp = z1;
  t.sp = 1;
  t.staged = 0;
  t.count = 0;
  t.visits = 0;
  t.paused = false;
  if (lane == 0) M.c.ring[0] = make_int2(0, 0);
  __builtin_amdgcn_wave_barrier();
}

// Drops the entries of a finished chunk [z0, zp) and moves z0 to zp.
__device__ __forceinline__ void trav_advance(WaveMem &M, int lane, Trav &t) {
  const uint64_t below = lanes_below(lane);
  int base = 0;
  for (int e0 = 0; e0 < t.count; e0 += 64) {
    const int e = e0 + lane;
    int id = 0;
    float tin = 0.0f, tout = 0.0f;
    bool keep = false;
    if (e < t.count) {
      id = M.l_id[e];
      tin = M.l_tin[e];
      tout = M.l_tout[e];
      keep = id >= t.zp;
    }
    __builtin_amdgcn_wave_barrier();
    const uint64_t b = ballot(keep);
    if (keep) {
      const int pos = base + __popcll(b & below);
      M.l_id[pos] = id;
      M.l_tin[pos] = tin;
      M.l_tout[pos] = tout;
    }
    base += __popcll(b);
    __builtin_amdgcn_wave_barrier();
  }
  t.count = base;
  t.z0 = t.zp;
  t.zp = t.z1;
  t.paused = false;
}

// Moves the staged leaves [head, staged) to the front; returns their number.
__device__ __forceinline__ int stage_front(WaveMem &M, int lane, int head, int staged) {
  const int rest = staged - head;
  for (int e0 = 0; e0 < rest; e0 += 64) {   // a write never passes an unread entry
    const int e = e0 + lane;
    const int v = e < rest ? M.c.st_id[head + e] : 0;
    __builtin_amdgcn_wave_barrier();
    if (e < rest) M.c.st_id[e] = v;
    __builtin_amdgcn_wave_barrier();
  }
  return rest;
}

// Runs (or resumes) the collection until it completes or pauses; sorts the
// finished chunk's entries into M.order and returns their number, or -1 on
// a malformed tree (error flag set).
__device__ __forceinline__ int trav_run(const SceneDev &s, WaveMem &M, const Ray &self, int lane, Trav &t,
                        int n_active, StatMem *stats, int32_t *err, int32_t &nodes_out,
                        int32_t &leaves_out, int64_t *cyc_excl) {
  if (n_active <= 0 || t.rays == 0 || t.z0 >= t.z1) {
    t.count = 0;
    t.sp = 0;
    t.staged = 0;
    return 0;
  }
  const int n_inner = n_active > 1 ? n_active - 1 : 1;
  const uint64_t rays = t.rays;
  const int z0 = t.z0;
  int z1 = t.z1;
  // stack S[0, sp): first leaf strictly decreasing towards the top S[sp-1]
  int sp = t.sp, staged = t.staged, count = t.count, visits = t.visits;
  const int visits0 = visits;
  const Cone cone = packet_cone(M, self, lane, rays);
  const uint64_t below = lanes_below(lane);
  for (;;) {
    __builtin_amdgcn_wave_barrier();
    // the frontier never grows past its end: a node adds at most three
    const int n = min(min(64, sp), min((kStageCap - staged) >> 2, max(1, (kRingCap - sp) / 3)));
    if (n > 0) {
      // four lanes to a node, one child each; 16 nodes at a time, all their
      // records requested before the first is tested
      const int child = lane & 3;
      vf4 q0[4], q1[4];
      bool live[4];
#pragma unroll
      for (int b = 0; b < 4; b++) {
        live[b] = false;
        if (16 * b >= n) continue;
        const int i = 16 * b + (lane >> 2);      // node 0 is the top (lowest Z)
        const int2 v = M.c.ring[max(sp - 1 - i, 0)];
        live[b] = (i < n) & (v.y < z1);          // else cut off by a later z1
        const vf4 *np = reinterpret_cast<const vf4 *>(s.quads) + (kQuadFloats / 4) * (live[b] ? v.x : 0) + 2 * child;
        q0[b] = np[0];
        q1[b] = np[1];
      }
      sp -= n;
      int link[4], first[4];
      uint64_t mI[4], mL[4], bad = 0;
      int totI = 0, totL = 0;
#pragma unroll
      for (int b = 0; b < 4; b++) {
        mI[b] = mL[b] = 0;
        link[b] = first[b] = 0;
        if (16 * b >= n) continue;
        visits += __popcll(ballot(live[b])) >> 2;
        link[b] = __float_as_int(q1[b].z);
        first[b] = __float_as_int(q1[b].w);      // an absent child's is past every range
        // the child's Z range ends where its right sibling's starts; the
        // last child's end is not stored, and its own children are tested
        const int nf = __builtin_amdgcn_update_dpp(0, first[b], 0xf9, 0xf, 0xf, false);
        const bool in = live[b] & (first[b] < z1) & ((child == 3) | (nf > z0)) &
                        ((link[b] >= 0) | (first[b] >= z0));
        // a malformed tree ends the walk; plain conjunctions, so that they
        // stay in lane masks instead of branching on every term
        bad |= ballot(in & ((first[b] < 0) |
                            (link[b] >= 0 ? link[b] >= n_inner : ~link[b] != first[b])));
        const bool hit = in & cone_box(cone, q0[b].x - self.ox, q0[b].y - self.oy, q0[b].z - self.oz,
                                       q0[b].w, q1[b].x, q1[b].y);
        mI[b] = ballot(hit & (link[b] >= 0));
        mL[b] = ballot(hit & (link[b] < 0));
        totI += __popcll(mI[b]);
        totL += __popcll(mL[b]);
      }
      if (visits > n_inner) { if (err) *err = 2; t.count = 0; t.sp = 0; t.staged = 0; return -1; }
      if (bad) { if (err) *err = 3; t.count = 0; t.sp = 0; t.staged = 0; return -1; }
      if (sp + totI > kRingCap) {
        // frontier overflow: lower z1 to keep half the pending subtrees
        int v[kRingCap / 64 + 4];
        bool ok[kRingCap / 64 + 4];
#pragma unroll
        for (int k = 0; k < kRingCap / 64; k++) {
          const int e = lane + 64 * k;
          ok[k] = e < sp;
          v[k] = ok[k] ? M.c.ring[e].y : 0;
        }
#pragma unroll
        for (int b = 0; b < 4; b++) {
          v[kRingCap / 64 + b] = first[b];
          ok[kRingCap / 64 + b] = (mI[b] >> lane) & 1ull;
        }
        z1 = select_cut(v, ok, z0 + 1, z1, kRingCap / 2);
        sp = compact_ring(M, lane, 0, sp, z1);
        totI = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          mI[b] &= ballot(first[b] < z1);
          totI += __popcll(mI[b]);
        }
      }
      // the children are below every entry left on the stack and, in batch
      // and lane order, ascending: the k-th of them goes to S[sp + totI - 1 - k];
      // leaves past a lowered z1 are filtered when tested
      int top = sp + totI - 1, end = staged;
#pragma unroll
      for (int b = 0; b < 4; b++) {
        if (16 * b >= n) continue;
        if ((mI[b] >> lane) & 1ull) M.c.ring[top - count_below(mI[b])] = make_int2(link[b], first[b]);
        if ((mL[b] >> lane) & 1ull) M.c.st_id[end + count_below(mL[b])] = first[b];
        top -= __popcll(mI[b]);
        end += __popcll(mL[b]);
      }
      sp += totI;
      staged += totL;
    }
    const bool done = sp == 0;
    // tests of staged leaves, 64 at a time, in staging order: the ellipsoid
    // (for a packet too wide, its bounding sphere) against the packet gives the
    // entry's depth bounds
    int head = 0;
    while (staged - head >= 64 || (done && staged > head)) {
      __builtin_amdgcn_wave_barrier();
      const int k = min(64, staged - head);
      if (count + k > kListCap) {
        // the list may overflow: pause at the smallest pending Z index if
        // the entries below it make a chunk
        int zq = sp > 0 ? M.c.ring[sp - 1].y : z1;
        for (int e = head + lane; e < staged; e += 64) zq = min(zq, M.c.st_id[e]);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) zq = min(zq, __shfl_xor(zq, o, 64));
        zq = min(__builtin_amdgcn_readfirstlane(zq), z1);
        int nb = 0;
        for (int e0 = 0; e0 < count; e0 += 64)
          nb += __popcll(ballot(e0 + lane < count && M.l_id[e0 + lane] < zq));
        if (nb > 0) {
          staged = stage_front(M, lane, head, staged);
          t.sp = sp; t.staged = staged; t.count = count; t.visits = visits; t.z1 = z1;
          t.zp = zq;
          t.paused = true;
          nodes_out += visits - visits0;
          return sort_list(M, lane, count, zq);
        }
      }
      int j = 0;
      bool test = false;
      if (lane < k) {
        j = M.c.st_id[head + lane];
        test = j < z1;
      }
      bool keep = false;
      float tmin = 0.0f, tmax = 0.0f;
      if (test) {
        // one 64-byte record a leaf, in one batch of loads
        const vf4 *np = reinterpret_cast<const vf4 *>(s.sup) + (kSupFloats / 4) * j;
        const vf4 m = np[0], n0 = np[1], n1 = np[2], n2 = np[3];
        pin_loaded(m); pin_loaded(n0); pin_loaded(n1); pin_loaded(n2);
        const float vx = m.x - self.ox, vy = m.y - self.oy, vz = m.z - self.oz;
        keep = cone.narrow ? cone_ellipsoid(cone, vx, vy, vz, n0, n1, n2, n0.w, m.w, &tmin,
                                             &tmax)
                           : cone_sphere(cone, vx, vy, vz, m.w, &tmin, &tmax);
      }
      if (stats && ballot(test)) {
        const int64_t c0 = clock64();
        // statistics only: AABB-only leaves per ray (box met, ellipsoid missed)
        const Gauss g = with_origin(load_gauss_lane(s.geom, test ? j : 0), self.ox, self.oy, self.oz);
        const float *bx = s.aabb + 6 * (size_t)(test ? j : 0);
        for (uint64_t rem = rays; rem; rem &= rem - 1) {
          const int r = __builtin_ctzll(rem);
          const Ray q = lds_ray(*stats, self, r);
          const float lo = M.rlo[r], hi = M.rhi[r];
          if (!test || !box_hit(bx[0], bx[1], bx[2], bx[3], bx[4], bx[5], q, lo, hi)) continue;
          const Chord ch = chord(g, q);
          if (!(ch.exists && ch.tin <= hi && ch.tout >= lo)) atomicAdd(&stats->cnt_box[r], 1);
        }
        if (cyc_excl) *cyc_excl += clock64() - c0;
      }
      leaves_out += k;
      int tot = __popcll(ballot(keep));
      if (count + tot > kListCap) {
        // list overflow: lower z1 so that half the list remains
        int v[kListCap / 64 + 1];
        bool ok[kListCap / 64 + 1];
#pragma unroll
        for (int q = 0; q < kListCap / 64; q++) {
          const int e = lane + 64 * q;
          ok[q] = e < count;
          v[q] = ok[q] ? M.l_id[e] : 0;
        }
        v[kListCap / 64] = j;
        ok[kListCap / 64] = keep;
        z1 = select_cut(v, ok, z0 + 1, z1, kListCap / 2);
        count = compact_list(M, lane, count, z1);
        keep = keep && j < z1;
        tot = __popcll(ballot(keep));
      }
      const uint64_t bk = ballot(keep);
      if (keep) {
        const int pos = count + __popcll(bk & below);
        M.l_id[pos] = j;
        M.l_tin[pos] = tmin;
        M.l_tout[pos] = tmax;
      }
      count += tot;
      head += k;
    }
    if (head > 0) staged = stage_front(M, lane, head, staged);
    if (done && staged == 0) break;
  }
  nodes_out += visits - visits0;
  t.sp = 0; t.staged = 0; t.count = count; t.visits = visits; t.z1 = z1;
  t.zp = z1;
  t.paused = false;
  return sort_list(M, lane, count, z1);
}

// ---------------------------------------------------------------------------
// Sources of a segment's candidate Gaussians, both in Z-index order: the
// window list (LDS) or every active Gaussian (brute force).

enum SourceKind { SRC_LIST = 0, SRC_BRUTE = 1 };

// Entries of M.order carry a mark bit above the slot index: set by a MARK
// pass for the entries some lane hit, read by a FILTER pass over the same
// list and the same segments.
constexpr int kOrderMark = 1 << 15;
enum CandMode { CAND_ALL = 0, CAND_MARK = 1, CAND_FILTER = 2 };

// Candidates are taken four at a time, and the ray direction in each one's
// frame, d' = M d, comes from the matrix cores (in the backward the SH colour
// sum_m f_m Y_m(d) too): the rows of a 16x16x4 FP32 product are 4 candidates x
// (3 components + 1 unused), its columns 16 of the tile's rays, its inner
// index 4 terms of the sum.  d' is one product per 16 rays, the colour four
// chained ones over the 16 coefficients.  Operand layout of
// v_mfma_f32_16x16x4_f32 (wave64): first operand X[i][k] in lane i + 16k,
// second Y[k][j] in lane j + 16k, D[i][j] in lane j + 16 (i / 4), register
// i % 4; so candidate q's three components for ray group g end in row q of the
// group's registers, and a 4x4 row transposition hands every lane (ray) its
// own values of the four candidates.  The unit adds the four products one
// after another in ascending k with one rounding each (measured bit for bit),
// so the values are those of the FMA chains fma(m_0, dx, fma(m_1, dy, m_2 dz))
// (terms in the order z, y, x) and f_0 Y_0 + f_1 Y_1 + ... .
//
// What bounds the loop is the SIMD's issue time, in which FP32 matrix
// instructions and vector instructions do not overlap (16000 of one take
// 0.245 ms, 128000 of the other 0.455 ms, both together 0.686 ms).  Measured
// per instruction with the SIMD full: 16x16x4 product 15.3 ns, row swap 3.4,
// readlane 1.85, FMA with a scalar operand 1.77, without 1.0.  d' of a
// candidate: 9 readlanes and 9 FMAs on them 32.6 ns, one product and three
// swaps 25.5 ns.  Its colour: 48 scalar-operand FMAs 85 ns and a scalar load's
// latency, against 71 ns with the operands loaded a group ahead -- but for
// every candidate.  In the forward with one lane a ray, where half the
// candidates are hit by no lane, the colour therefore stays with the vector
// units (a split forward's operands serve 2 or 4 times as few groups, and it
// takes the matrix units); the backward's
// candidates are the hit ones.  1M Gaussians, 4 x 1024x768: forward 41.5 ->
// 39.7 ms (43.2 with the colour here too), backward 32.4 -> 30.3 ms (with sum_rows16).
template <int S>
struct TileOps {
  static constexpr int kGroups = 4 / S;   // ray groups of 16
  float d[kGroups];      // direction operand of rays 16g .. 16g + 15: k = 0, 1, 2 -> z, y, x; 3 -> 0
  float y[kGroups][4];   // basis operand, [ray group][4 coefficients 4q .. 4q + 3] (COL)
};

template <bool COL, int S>
__device__ __forceinline__ void tile_ops(TileOps<S> &o, const Ray &r, const float *Y, int lane) {
  const int k = lane >> 4;
#pragma unroll
  for (int g = 0; g < TileOps<S>::kGroups; g++) {
    const int src = 16 * g + (lane & 15);
    const float x = __shfl(r.dx, src, 64), y = __shfl(r.dy, src, 64), z = __shfl(r.dz, src, 64);
    o.d[g] = k == 0 ? z : k == 1 ? y : k == 2 ? x : 0.0f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      if constexpr (!COL) break;
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; e++) t[e] = __shfl(Y[4 * q + e], src, 64);
      o.y[g][q] = k == 0 ? t[0] : k == 1 ? t[1] : k == 2 ? t[2] : t[3];
    }
  }
}

// One candidate that some lane of the wave hit, as the segment loops see it:
// the lane's chord and colour, and (pass B) its ray in the local frame.
struct Cand {
  float k2, l2sig;          // uniform
  Chord ch;
  float ox, oy, oz;         // uniform
  float ex, ey, ez;         // uniform: camera centre minus mean
  float dx, dy, dz;
  float cr, cg, cb;
};

// A lane's matrix operands of a group of four candidates.
struct CandOps {
  float m;       // lane (row 4c + i, k): M_c[i][2 - k]
  vf4 f;         // lane (row 4c + i, k): coefficients 4q + k, q = 0..3, of channel i
};

// Issues the operand loads of a lane's candidate of the group (`mine`: that of
// row c of its operands, c = (lane >> 2) & 3).
template <bool COL>
__device__ __forceinline__ CandOps cand_fetch(const SceneDev &s, uint32_t mine, int lane) {
  const int i = min(lane & 3, 2), k = lane >> 4;
  CandOps G;
  // (32-bit byte offsets: at most 2^23 records of 192 bytes)
  const uint32_t mo = mine * (4u * kGeomFloats) + 4u * (uint32_t)(G_M + 3 * i + 2 - min(k, 2));
  G.m = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(s.geom) + mo);
  if (COL) {
    const uint32_t fo = mine * (4u * kColFloats) + 4u * (uint32_t)(16 * i + 4 * k);
    G.f = *reinterpret_cast<const vf4 *>(reinterpret_cast<const char *>(s.col) + fo);
  }
  return G;
}
template <bool COL>
__device__ __forceinline__ void cand_pin(const CandOps &G) {
  pin_lane(__float_as_uint(G.m));
  if (COL) pin_loaded(G.f);
}

// Calls fn(c, j, g, hit) for every candidate j (the c-th of its group of four,
// a constant in each inlined copy) whose chord meets [lo, hi] in some lane
// with `want` set; `hit` says in which lanes, g is its Cand (colour left out
// unless COL).  visit() runs once per candidate tested (statistics).
// `a_min`/`b_max` bound the live lanes' segments for the list's uniform
// depth pre-check.  List entries are taken 64 at a time: lane i holds entry
// base + i and loads that entry's geometry, so one memory round trip serves
// the whole block; the surviving candidates then go through in groups of
// four, the next group's operand loads in flight meanwhile.  A group's four
// chords are one branch-free run of vector work, so that the four dependent
// chains (with a reciprocal and a square root each) overlap; the colour's
// matrix instructions are spread through it.
// after(ids, first, hits) runs once per group when the next operands have
// arrived (candidate c is lane first + c of `ids`, bit c of `hits` says whether
// some lane hit it): memory operations that count against the same counter
// (atomics) belong there, or the wait for the loads would wait for them too.
// CAND_MARK: a visited entry's mark is set to whether some lane hit it.  With
// use_marks, a CAND_MARK pass trusts the marks already set (from a record of
// the same pass) and visits only the marked entries, and a CAND_FILTER pass
// visits only the marked entries (list source only; the brute-force source
// visits everything).
// LATE: the colour's matrix instructions follow the hit tests, in groups some
// lane hit, instead of going in between the chords.
template <int MODE, bool COL, bool LATE = false, int S, class Visit, class Fn, class After>
__device__ __forceinline__ void for_each_candidate(int kind, const SceneDev &s, ListMem &M,
                                                   int count, int lane, float a_min, float b_max,
                                                   int n_active, const Ray &r, const TileOps<S> &ops,
                                                   bool want, float lo, float hi, Visit &&visit,
                                                   Fn &&fn, After &&after, bool use_marks = false) {
  const bool list = kind == SRC_LIST;
  const int total = list ? count : n_active;
  const uint64_t wanted = ballot(want);
  for (int base = 0; base < total; base += 64) {
    const int e = base + lane;
    int id = 0, o = 0;
    bool keep = false;
    if (e < total) {
      if (list) {
        const int om = M.order[e];
        o = om & (kOrderMark - 1);
        // the entry's three words are read together (no short-circuit
        // between the depth tests, which would wait for each read in turn)
        const float tin = M.l_tin[o], tout = M.l_tout[o];
        id = M.l_id[o];
        keep = !(tin > b_max) & !(tout < a_min);
        if (MODE != CAND_ALL) keep = keep & (!use_marks | ((om & kOrderMark) != 0));
      } else {
        id = e;
        keep = true;
      }
    }
    const uint64_t kept = ballot(keep);
    if (!kept) continue;
    const int n = __popcll(kept), rank = __popcll(kept & lanes_below(lane));
    // the block's candidates move to lanes 0 .. n - 1, in order
    if (keep) M.cand[rank] = id;
    __builtin_amdgcn_wave_barrier();
    const uint32_t first_of = (uint32_t)M.cand[min((lane >> 2) & 3, n - 1)];
    const int cid = M.cand[min(lane, n - 1)];
    __builtin_amdgcn_wave_barrier();
    CandOps cur = cand_fetch<COL>(s, first_of, lane);
    const Gauss mine = with_origin(load_gauss_lane(s.geom, cid), r.ox, r.oy, r.oz);
    int next_id = __shfl(cid, 4 + ((lane >> 2) & 3), 64);
    cand_pin<COL>(cur);
    uint64_t hits = 0;   // (uniform) the block's candidates some lane hit
    for (int first = 0; first < n; first += 4) {
      // d' of the group's candidates, transposed to the lanes; the next
      // group's loads and the readlanes run beside the matrix instructions
      constexpr int kG = TileOps<S>::kGroups;
      f4v acc[kG];
      const float mm = lane < 48 ? cur.m : 0.0f;
#pragma unroll
      for (int g = 0; g < kG; g++) {
        const f4v z = {0.0f, 0.0f, 0.0f, 0.0f};
        acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(mm, ops.d[g], z, 0, 0, 0);
      }
      const CandOps nxt = cand_fetch<COL>(s, (uint32_t)next_id, lane);
      Cand g[4];
#pragma unroll
      for (int c = 0; c < 4; c++) {
        g[c].ox = uniform_lane(mine.ox, first + c);
        g[c].oy = uniform_lane(mine.oy, first + c);
        g[c].oz = uniform_lane(mine.oz, first + c);
        g[c].k2 = uniform_lane(mine.k2, first + c);
        g[c].l2sig = uniform_lane(mine.l2sig, first + c);
        if constexpr (MODE == CAND_FILTER) {   // (pass B)
          g[c].ex = uniform_lane(r.ox - mine.mx, first + c);
          g[c].ey = uniform_lane(r.oy - mine.my, first + c);
          g[c].ez = uniform_lane(r.oz - mine.mz, first + c);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      next_id = __shfl(cid, first + 8 + ((lane >> 2) & 3), 64);
      {
        float d[3][4];
#pragma unroll
        for (int i = 0; i < 3; i++) {
#pragma unroll
          for (int q = 0; q < 4; q++) d[i][q] = acc[q % kG][i];
          transpose_rows(d[i]);
        }
#pragma unroll
        for (int c = 0; c < 4; c++) { g[c].dx = d[0][c]; g[c].dy = d[1][c]; g[c].dz = d[2][c]; }
      }
      // the four chords (chord_local, step by step), one of the colour's 16
      // matrix instructions before every few vector ones; the barriers keep
      // the order, which the compiler's scheduler would undo
      if constexpr (COL) {
#pragma unroll
        for (int p = 0; p < kG; p++) acc[p] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
      }
      auto mm_step = [&](int i) {   // (16 steps; every S-th carries an instruction)
        if constexpr (COL && !LATE) {
          if (i % S == 0) {
            const int q = i / 4, p = (i / S) % kG;
            __builtin_amdgcn_sched_barrier(0);
            acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.f[q], ops.y[p][q], acc[p], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      };
      float B[4], rA[4], x[4], w[4];
#pragma unroll
      for (int c = 0; c < 4; c++) {
        if (!(c & 1)) mm_step(c >> 1);
        g[c].ch.A = fmaf(g[c].dx, g[c].dx, fmaf(g[c].dy, g[c].dy, g[c].dz * g[c].dz));
      }
#pragma unroll
      for (int c = 0; c < 4; c++) {
        if (!(c & 1)) mm_step(2 + (c >> 1));
        rA[c] = __builtin_amdgcn_rcpf(g[c].ch.A);
        B[c] = fmaf(g[c].ox, g[c].dx, fmaf(g[c].oy, g[c].dy, g[c].oz * g[c].dz));
      }
      mm_step(4);
#pragma unroll
      for (int c = 0; c < 4; c++) g[c].ch.ts = -B[c] * rA[c];
#pragma unroll
      for (int c = 0; c < 4; c++) {
        mm_step(5 + c);
        const float px = fmaf(g[c].ch.ts, g[c].dx, g[c].ox), py = fmaf(g[c].ch.ts, g[c].dy, g[c].oy),
                    pz = fmaf(g[c].ch.ts, g[c].dz, g[c].oz);
        g[c].ch.h2 = fmaf(px, px, fmaf(py, py, pz * pz));
      }
      mm_step(9);
#pragma unroll
      for (int c = 0; c < 4; c++) x[c] = fmaxf(g[c].k2 - g[c].ch.h2, 0.0f);
      mm_step(10);
#pragma unroll
      for (int c = 0; c < 4; c++) w[c] = __builtin_amdgcn_sqrtf(x[c] * rA[c]);
      mm_step(11);
      uint64_t any[4];
#pragma unroll
      for (int c = 0; c < 4; c++) {
        g[c].ch.tin = g[c].ch.ts - w[c];
        g[c].ch.tout = g[c].ch.ts + w[c];
        // lane masks, not a chain of short-circuit branches
        any[c] = ballot(g[c].ch.h2 <= g[c].k2) & ballot(g[c].ch.tin <= hi) &
                 ballot(g[c].ch.tout >= lo) & (first + c < n ? wanted : 0ull);
        mm_step(12 + c);
      }
      float col[3][4] = {};
      if (COL && (!LATE || (any[0] | any[1] | any[2] | any[3]) != 0)) {
        if constexpr (LATE) {
#pragma unroll
          for (int q = 0; q < 4; q++)
#pragma unroll
            for (int p = 0; p < kG; p++)
              acc[p] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.f[q], ops.y[p][q], acc[p], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 3; i++) {
#pragma unroll
          for (int q = 0; q < 4; q++) col[i][q] = acc[q % kG][i];
          transpose_rows(col[i]);
        }
      }
#pragma unroll
      for (int c = 0; c < 4; c++) {
        if (first + c < n) visit();
        if (any[c] != 0) {
          if (MODE == CAND_MARK) hits |= 1ull << (first + c);
          if constexpr (COL) { g[c].cr = col[0][c]; g[c].cg = col[1][c]; g[c].cb = col[2][c]; }
          fn(c, __builtin_amdgcn_readlane(cid, first + c), g[c],
             __builtin_amdgcn_inverse_ballot_w64(any[c]));
        }
      }
      cand_pin<COL>(nxt);
      after(cid, first, (any[0] != 0 ? 1u : 0u) | (any[1] != 0 ? 2u : 0u) | (any[2] != 0 ? 4u : 0u) |
                            (any[3] != 0 ? 8u : 0u));
      cur = nxt;
    }
    if (MODE == CAND_MARK && list && !use_marks && keep)
      M.order[e] = (uint16_t)(o | (((hits >> rank) & 1ull) ? kOrderMark : 0));
  }
}

// Window-list record of a tile (layout next to kWrecHeader): a forward
// appends every collection's sorted chunk with the collection state its
// callers read, and after every pass over a list the marks of the entries
// some lane hit; a backward of the same rays reads them back in the same
// order instead of walking the tree, and visits only the marked entries.
// Every record starts with the offset of the tile's next record.
struct WinRec {
  uint32_t *slot = nullptr;   // the tile's (complete, first record) pair
  uint32_t cur = kWrecNone;   // replay: next record to read; record: last record written
  uint32_t share = 0;         // record: share of the pool its records come from
  bool ok = false;            // record: nothing dropped so far; replay: tile complete
};

// FORWARD: to be recorded if the options say so; else to be replayed.
template <bool FORWARD>
__device__ __forceinline__ void rec_start(WinRec &R, const MarchOpts &op, const ViewTable &vt,
                                          int w) {
  R.slot = op.replay_mode ? op.wrec_tile + 2 * (size_t)(vt.tile0 + w) : nullptr;
  R.cur = kWrecNone;
  R.ok = false;
  if (FORWARD && op.replay_mode == 1) {
    R.ok = true;
    R.share = (uint32_t)(vt.tile0 + w) & (op.wrec_shares - 1);
    if (__lane_id() == 0) R.slot[1] = kWrecNone;
  } else if (!FORWARD && op.replay_mode == 2) {
    R.ok = uniform_int((int)R.slot[0]) == 1;
    R.cur = (uint32_t)uniform_int((int)R.slot[1]);
  }
}

// forward: the tile's status once all its records are in
__device__ __forceinline__ void rec_finish(WinRec &R, const MarchOpts &op, int lane) {
  if (op.replay_mode != 1) return;
  if (lane == 0) R.slot[0] = R.ok ? 1u : 0u;
}

// Appends a record of `size` dwords to the tile's chain; kWrecNone (and the
// tile marked incomplete) when the pool is full.
__device__ __forceinline__ uint32_t rec_alloc(WinRec &R, const MarchOpts &op, uint32_t size,
                                              int lane) {
  uint64_t at = 0;
  for (uint32_t tries = 0;; tries++) {
    if (tries == op.wrec_shares) {
      if (lane == 0) op.wrec[kWrecFull] = 1u;
      R.ok = false;
      return kWrecNone;
    }
    // a 64-bit counter: failed allocations keep adding to it, and it must not
    // wrap back into the share
    unsigned long long got = 0;
    if (lane == 0)
      got = atomicAdd(reinterpret_cast<unsigned long long *>(op.wrec + kWrecLine * R.share), (unsigned long long)size);
    at = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(got >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)got);
    if (at + size <= op.wrec_len) break;
    R.share = (R.share + 1) & (op.wrec_shares - 1);
  }
  const uint32_t off = (uint32_t)kWrecLine * op.wrec_shares + op.wrec_len * R.share + (uint32_t)at;
  if (lane == 0) {
    op.wrec[off] = kWrecNone;
    // link from the previous record, or the tile's slot
    uint32_t *from = R.cur != kWrecNone ? op.wrec + R.cur : R.slot + 1;
    *from = off;
  }
  R.cur = off;
  return off;
}

// Checks that a record of at least `size` dwords at `off` lies in the pool.
__device__ __forceinline__ bool rec_fits(const MarchOpts &op, uint32_t off, uint64_t size) {
  return off < op.wrec_cap && (uint64_t)off + size <= op.wrec_cap;
}

__device__ __forceinline__ void rec_put(WinRec &R, const MarchOpts &op, const ListMem &M,
                                        const Trav &t, int cnt, int lane) {
  if (!R.ok) return;
  const int n = cnt > 0 ? cnt : 0;
  const uint32_t off = rec_alloc(R, op, kWrecHeader + 3 * n, lane);
  if (off == kWrecNone) return;
  uint32_t *p = op.wrec + off;
  if (lane == 0) {
    p[1] = (uint32_t)cnt; p[2] = t.paused ? 1u : 0u; p[3] = (uint32_t)t.z0;
    p[4] = (uint32_t)t.z1; p[5] = (uint32_t)t.zp; p[6] = (uint32_t)t.count;
  }
  for (int e = lane; e < n; e += 64) {
    const int o = M.order[e] & (kOrderMark - 1);
    p[kWrecHeader + 3 * e] = (uint32_t)M.l_id[o];
    p[kWrecHeader + 3 * e + 1] = __float_as_uint(M.l_tin[o]);
    p[kWrecHeader + 3 * e + 2] = __float_as_uint(M.l_tout[o]);
  }
}

// The marks of the current list's `count` entries after a pass: [next, count,
// then one 64-bit ballot per 64 entries].
__device__ __forceinline__ void rec_put_marks(WinRec &R, const MarchOpts &op, const ListMem &M,
                                              int count, int lane) {
  if (!R.ok) return;
  const int words = (count + 63) >> 6;
  const uint32_t off = rec_alloc(R, op, 2 + 2 * words, lane);
  if (off == kWrecNone) return;
  uint32_t *p = op.wrec + off;
  if (lane == 0) p[1] = (uint32_t)count;
  for (int q = 0; q < words; q++) {
    const int e = 64 * q + lane;
    const uint64_t b = ballot(e < count && (M.order[e] & kOrderMark) != 0);
    if (lane == 0) {
      p[2 + 2 * q] = (uint32_t)b;
      p[3 + 2 * q] = (uint32_t)(b >> 32);
    }
  }
}

// The per-sample sums of a segment step (layout next to kSrecHeader): lanes
// `hit` store sigma_k and W_k, lanes `empty` their restart distance.
template <int NS>
__device__ __forceinline__ void rec_put_samples(WinRec &R, const MarchOpts &op, bool hit,
                                                bool empty, float best, const float *sg,
                                                const float *W0, const float *W1,
                                                const float *W2, int lane) {
  if (!R.ok) return;
  const uint64_t hm = ballot(hit), em = ballot(empty);
  const int nh = __popcll(hm), ne = __popcll(em);
  const uint32_t off = rec_alloc(R, op, kSrecHeader + 4 * NS * nh + ne, lane);
  if (off == kWrecNone) return;
  uint32_t *p = op.wrec + off;
  if (lane == 0) {
    p[1] = (uint32_t)hm; p[2] = (uint32_t)(hm >> 32);
    p[3] = (uint32_t)em; p[4] = (uint32_t)(em >> 32);
  }
  float *q = reinterpret_cast<float *>(p + kSrecHeader);
  const uint64_t below = lanes_below(lane);
  if (hit) {
    const int rk = __popcll(hm & below);
#pragma unroll
    for (int k = 0; k < NS; k++) {
      q[(4 * k) * nh + rk] = sg[k];
      q[(4 * k + 1) * nh + rk] = W0[k];
      q[(4 * k + 2) * nh + rk] = W1[k];
      q[(4 * k + 3) * nh + rk] = W2[k];
    }
  }
  if (empty) q[4 * NS * nh + __popcll(em & below)] = best;
}

// Reads the sample record of a segment step back: sigma_k into sg, G . W_k
// into GW, and for an empty segment the restart distance into *best.
// Returns whether this lane's segment hit something.  A record that does not
// match the lanes that march (cannot happen) is reported, and its lanes read
// as empty with no restart.
template <int NS>
__device__ __forceinline__ bool rec_get_samples(WinRec &R, const MarchOpts &op, bool go, float Gc0,
                                                float Gc1, float Gc2, float *sg, float *GW,
                                                float *best, int lane, int32_t *err) {
  *best = kInf;
  const uint32_t off = R.cur;
  if (off == kWrecNone || !rec_fits(op, off, kSrecHeader)) {
    if (err) *err = 5;
    R.cur = kWrecNone;
    return false;
  }
  const uint32_t *p = op.wrec + off;
  // the header's five words in one batch of loads
  uint32_t hw[kSrecHeader];
#pragma unroll
  for (int i = 0; i < kSrecHeader; i++) hw[i] = p[i];
#pragma unroll
  for (int i = 0; i < kSrecHeader; i++) pin_lane(hw[i]);
  const uint64_t hm = ((uint64_t)(uint32_t)uniform_int((int)hw[2]) << 32) | (uint32_t)uniform_int((int)hw[1]);
  const uint64_t em = ((uint64_t)(uint32_t)uniform_int((int)hw[4]) << 32) | (uint32_t)uniform_int((int)hw[3]);
  const int nh = __popcll(hm), ne = __popcll(em);
  if ((hm | em) != ballot(go) || (hm & em) != 0 ||
      !rec_fits(op, off, kSrecHeader + 4 * (uint64_t)NS * nh + ne)) {
    if (err) *err = 5;
    R.cur = kWrecNone;
    return false;
  }
  R.cur = (uint32_t)uniform_int((int)hw[0]);
  const float *q = reinterpret_cast<const float *>(p + kSrecHeader);
  const uint64_t below = lanes_below(lane);
  const bool hit = (hm >> lane) & 1ull;
  if (hit) {
    const int rk = __popcll(hm & below);
    // the 4 N_s values in one batch of loads (the compiler would otherwise
    // wait for every few of them in turn to keep fewer registers live)
    float v[4 * NS];
#pragma unroll
    for (int i = 0; i < 4 * NS; i++) v[i] = q[i * nh + rk];
#pragma unroll
    for (int i = 0; i < 4 * NS; i++) pin_lane(__float_as_uint(v[i]));
#pragma unroll
    for (int k = 0; k < NS; k++) {
      sg[k] = v[4 * k];
      GW[k] = fmaf(Gc0, v[4 * k + 1], fmaf(Gc1, v[4 * k + 2], Gc2 * v[4 * k + 3]));
    }
  }
  if ((em >> lane) & 1ull) *best = q[4 * NS * nh + __popcll(em & below)];
  return hit;
}

// Loads the chunk at pool offset `off` into the list (identity order, no
// marks); returns its collection's result and the next record in *next.
__device__ __forceinline__ int rec_load(const MarchOpts &op, ListMem &M, uint32_t off, int lane,
                                        uint32_t *next) {
  // a record always fits the pool and the list; anything else is reported
  if (!rec_fits(op, off, kWrecHeader)) { *next = kWrecNone; return -1; }
  const uint32_t *p = op.wrec + off;
  const int cnt = uniform_int((int)p[1]);
  const int n = cnt > 0 ? cnt : 0;
  if (n > kListCap || !rec_fits(op, off, kWrecHeader + 3 * (uint64_t)n)) {
    *next = kWrecNone;
    return -1;
  }
  __builtin_amdgcn_wave_barrier();
  for (int e = lane; e < n; e += 64) {
    M.l_id[e] = (int)p[kWrecHeader + 3 * e];
    M.l_tin[e] = __uint_as_float(p[kWrecHeader + 3 * e + 1]);
    M.l_tout[e] = __uint_as_float(p[kWrecHeader + 3 * e + 2]);
    M.order[e] = (uint16_t)e;
  }
  __builtin_amdgcn_wave_barrier();
  *next = (uint32_t)uniform_int((int)p[0]);
  return cnt;
}

// Sets the list's marks from the marks record at `off` (which must cover
// `count` entries); false on a broken record.
__device__ __forceinline__ bool rec_load_marks(const MarchOpts &op, ListMem &M, uint32_t off,
                                               int count, int lane, uint32_t *next) {
  const int words = (count + 63) >> 6;
  if (!rec_fits(op, off, 2 + 2 * (uint64_t)words)) { *next = kWrecNone; return false; }
  const uint32_t *p = op.wrec + off;
  const uint32_t h0 = p[0], h1 = p[1];
  pin_lane(h0); pin_lane(h1);
  constexpr int kSlots = kListCap / 64;
  if (uniform_int((int)h1) != count || words > kSlots) { *next = kWrecNone; return false; }
  __builtin_amdgcn_wave_barrier();
  if (words > 0) {
    // every mark word in one batch of loads (slots past the end read the
    // last word again and are not used)
    uint32_t w[kSlots];
#pragma unroll
    for (int q = 0; q < kSlots; q++) w[q] = p[2 + 2 * min(q, words - 1) + (lane >> 5)];
#pragma unroll
    for (int q = 0; q < kSlots; q++) pin_lane(w[q]);
#pragma unroll
    for (int q = 0; q < kSlots; q++) {
      const int e = 64 * q + lane;
      if (q < words && e < count) {
        const int o = M.order[e] & (kOrderMark - 1);
        M.order[e] = (uint16_t)(o | (((w[q] >> (lane & 31)) & 1u) ? kOrderMark : 0));
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
  *next = (uint32_t)uniform_int((int)h0);
  return true;
}

// Backward pass over the current list: in a replayed tile, the forward's
// marks of this pass (true: visit only those), else false (mark as it goes).
__device__ __forceinline__ bool rec_next_marks(WinRec &R, const MarchOpts &op, ListMem &M,
                                               int count, int kind, int lane, int32_t *err) {
  if (!(op.replay_mode == 2 && R.ok) || kind != SRC_LIST) return false;
  uint32_t next;
  if (R.cur == kWrecNone || !rec_load_marks(op, M, R.cur, count, lane, &next)) {
    // a broken record (cannot happen): flag it; later reads of this tile's
    // record find no next record and end its rays
    if (err) *err = 5;
    R.cur = kWrecNone;
    return false;
  }
  R.cur = next;
  return true;
}

// One collection: the tree walk (recorded in a recording forward) or, in a
// replaying backward of a complete tile, the recorded chunk and state.
// *start receives the chunk's record offset.
// A forward (WIN_SEARCH) never reads a record and a replaying backward
// (WIN_REPLAY) never walks the tree: the other branch is compiled out, as its
// registers would count against the whole kernel.
enum WinMode { WIN_SEARCH = 0, WIN_BOTH, WIN_REPLAY };
template <int MODE, class Mem>
__device__ __forceinline__ int collect(const SceneDev &s, const MarchOpts &op, Mem &M,
                                       const Ray &r, int lane, Trav &t, int n_active, StatMem *stats,
                                       int32_t *err, int32_t &nodes, int32_t &leaves,
                                       int64_t *cyc_excl, WinRec &R, uint32_t *start) {
  if (MODE == WIN_REPLAY || (MODE == WIN_BOTH && op.replay_mode == 2 && R.ok)) {
    if (R.cur == kWrecNone || !rec_fits(op, R.cur, kWrecHeader)) {   // a broken record
      if (err) *err = 5;
      t.count = 0;
      t.paused = false;
      return -1;
    }
    const uint32_t *p = op.wrec + R.cur;
    t.paused = uniform_int((int)p[2]) != 0;
    t.z0 = uniform_int((int)p[3]);
    t.z1 = uniform_int((int)p[4]);
    t.zp = uniform_int((int)p[5]);
    t.count = uniform_int((int)p[6]);
    *start = R.cur;
    uint32_t next;
    const int cnt = rec_load(op, M, R.cur, lane, &next);
    if (cnt < 0 && err) *err = 5;
    R.cur = next;
    return cnt;
  }
  int cnt = -1;
  if constexpr (MODE != WIN_REPLAY) {
    // the walk is a chain of dependent loads and short bursts of work: while
    // it runs, the wave's instructions issue ahead of other waves' long
    // arithmetic runs on the same SIMD (wave priority, not a queue priority)
    __builtin_amdgcn_s_setprio(3);
    cnt = trav_run(s, M, r, lane, t, n_active, stats, err, nodes, leaves, cyc_excl);
    __builtin_amdgcn_s_setprio(0);
    if (op.replay_mode == 1) rec_put(R, op, M, t, cnt, lane);
    *start = R.cur;
  }
  return cnt;
}

// Per-wave window bookkeeping shared by forward and backward.
struct Window {
  float len, len_min, len_max;   // uniform window length beyond the segment, and its bounds
  bool valid;                    // per lane: the current list covers this lane's later segments
  float hi;                      // per lane window end
  int count;                     // uniform number of candidates in M.order
  int kind;                      // SourceKind of the current candidates
  bool chunked;                  // uniform: this segment's candidates come in Z chunks
  int zend;                      // uniform end of the Z range the chunks cover
  uint32_t rec_first, rec_last;  // record offsets of the segment's first and last chunk
  Trav t;                        // the collection behind the list
};

// Makes sure every live lane whose segment fits its window can march; when
// no live lane can, collects a new window for all live lanes.  A window that
// could not be collected whole serves the current segment only, chunk by
// chunk.
template <int MODE, class Mem>
__device__ __forceinline__ void ensure_window(const SceneDev &s, const MarchOpts &op, Mem &M,
                                              const Ray &r, int lane, int n_active, bool alive,
                                              float a, float b, Window &w, StatMem *stats,
                                              int32_t *err, int32_t &nodes, int32_t &leaves,
                                              int32_t &windows, bool &fits, WinRec &R,
                                              int64_t *cyc_excl = nullptr) {
  if (MODE != WIN_REPLAY && op.brute_force) {
    w.kind = SRC_BRUTE;
    w.chunked = false;
    fits = alive;
    return;
  }
  fits = alive && w.valid && b <= w.hi;
  if (ballot(fits) != 0 || ballot(alive) == 0) {
    w.chunked = false;
    return;
  }
  const uint64_t rays = ballot(alive);
  const float hi = alive ? fmaxf(a + w.len, b) : -kInf;
  if constexpr (MODE != WIN_REPLAY) {
    M.rlo[lane] = alive ? a : kInf;
    M.rhi[lane] = hi;
    windows++;
    trav_start(M, lane, w.t, rays, 0, n_active);
  }
  w.zend = n_active;
  const int cnt = collect<MODE>(s, op, M, r, lane, w.t, n_active, stats, err, nodes, leaves,
                                  cyc_excl, R, &w.rec_first);
  w.rec_last = w.rec_first;
  w.kind = SRC_LIST;
  w.count = cnt > 0 ? cnt : 0;   // a malformed tree ends the rays (error flag set)
  w.chunked = cnt >= 0 && (w.t.paused || w.t.z1 < n_active);
  if (!w.chunked) {
    w.valid = alive;
    w.hi = hi;
    if (w.t.count < kListCap / 4) w.len = fminf(fmaxf(w.len * 1.5f, w.len_min), w.len_max);
  } else {
    w.valid = false;
    w.len = w.len * 0.5f < w.len_min ? 0.0f : w.len * 0.5f;
    // the chunks to come serve this segment only: what is left of the walk
    // needs no longer window (3M Gaussians, camera inside the dense part, an
    // initial window of four segments: 17.8k -> 11.6k leaf tests a tile,
    // forward 28.3 -> 23.7 ms)
    if constexpr (MODE != WIN_REPLAY) M.rhi[lane] = alive ? b : -kInf;
  }
  fits = alive;
}

// Starts the chunks of the current segment again over the Z range [0, zend),
// for the lanes in `lanes` over their segments [a, b].
__device__ __forceinline__ void first_chunk(const SceneDev &s, WaveMem &M, const Ray &r, int lane,
                                            int n_active, bool lanes, float a, float b, int zend,
                                            Window &w, StatMem *stats, int32_t *err, int32_t &nodes,
                                            int32_t &leaves, int32_t &windows) {
  const uint64_t rays = ballot(lanes);
  M.rlo[lane] = lanes ? a : kInf;
  M.rhi[lane] = lanes ? b : -kInf;
  windows++;
  trav_start(M, lane, w.t, rays, 0, zend);
  w.zend = zend;
  const int cnt = trav_run(s, M, r, lane, w.t, n_active, stats, err, nodes, leaves, nullptr);
  w.count = cnt > 0 ? cnt : 0;
}

// In chunked mode, moves to the candidates of the next Z chunk: resumes a
// paused collection, or after a cut at z1 collects again from z1 for the
// lanes in `lanes` over their segments [a, b].  False when the segment's
// candidates are exhausted.
template <int MODE, class Mem>
__device__ __forceinline__ bool next_chunk(const SceneDev &s, const MarchOpts &op, Mem &M,
                                           const Ray &r, int lane, int n_active, bool lanes,
                                           float a, float b, Window &w, StatMem *stats, int32_t *err,
                                           int32_t &nodes, int32_t &leaves, int32_t &windows,
                                           WinRec &R, int64_t *cyc_excl = nullptr) {
  if (!w.chunked) return false;
  if (w.t.paused) {
    if constexpr (MODE != WIN_REPLAY)
      if (!(MODE == WIN_BOTH && op.replay_mode == 2 && R.ok)) trav_advance(M, lane, w.t);
  } else {
    if (w.t.z1 >= w.zend) return false;
    const uint64_t rays = ballot(lanes);
    if (rays == 0) return false;
    if constexpr (MODE != WIN_REPLAY) {
      M.rlo[lane] = lanes ? a : kInf;
      M.rhi[lane] = lanes ? b : -kInf;
      windows++;
      trav_start(M, lane, w.t, rays, w.t.z1, w.zend);
    }
  }
  const int cnt = collect<MODE>(s, op, M, r, lane, w.t, n_active, stats, err, nodes, leaves,
                                  cyc_excl, R, &w.rec_last);
  if (cnt < 0) {
    w.count = 0;
    w.chunked = false;
    return false;
  }
  w.count = cnt;
  return true;
}

// ---------------------------------------------------------------------------
// Forward kernel (and the hit-dump variant).

template <int NS, int S, bool DUMP, bool STATS, bool SG = false>
__global__ __launch_bounds__(kWave, NS / S <= 8 ? 3 : 2) void k_forward(SceneDev s, ViewTable vt, MarchOpts op,
                                                   FwdOut out, LaunchShape ls) {
  __shared__ WaveMem M;
  __shared__ StatMemOf<STATS> SM;
  StatMem *sm = nullptr;
  if constexpr (STATS) sm = &SM;
  constexpr int kRays = 64 / S, NL = NS / S;   // rays of the tile; samples of a ray per lane
  const int lane = threadIdx.x;
  const int sub = lane / kRays;                // this lane's samples: sub, sub + S, ...
  const int n_active = uniform_int(s.counters[0]);
  const bool grid = !op.adaptive && op.ess != 2;
  constexpr bool stats = STATS;
  if (!DUMP && !marches_any(s, op, vt)) return;
  bool first = true;
  for (;;) {
    int w;
    if (op.persistent) {
      w = pop_tile(ls.queue, vt.n_tiles, blockIdx.x & 7, lane);
      if (w < 0) break;
    } else {
      if (!first) break;
      w = xcd_block(blockIdx.x, gridDim.x);
      if (w >= vt.n_tiles) break;
    }
    first = false;

    Pixel px;
    int dump_slot = 0;
    if (DUMP) {
      dump_slot = w * 64 + lane;
      px.view = 0;
      px.valid = dump_slot < out.dump_n;
      const int pix = px.valid ? out.dump_pix[dump_slot] : 0;
      px.px = pix % vt.v[0].width;
      px.py = pix / vt.v[0].width;
      px.ray = dump_slot;
    } else {
      px = tile_pixel(vt, op, w, lane & (kRays - 1), kRays);
    }
    const View &V = vt.v[px.view];
    if (!DUMP && !marches_view(s, op, V)) continue;
    const Ray r = make_ray(V, px.px, px.py);
    if constexpr (STATS) {
      sm->rdx[lane] = r.dx; sm->rdy[lane] = r.dy; sm->rdz[lane] = r.dz;
      sm->rix[lane] = r.ix; sm->riy[lane] = r.iy; sm->riz[lane] = r.iz;
      sm->cnt_box[lane] = 0;
    }
    const float tn = V.t_near, tf = V.t_far;
    float Y[16];
    sh_basis(op.sh_k, r.dx, r.dy, r.dz, Y);
    TileOps<S> ops;
    tile_ops<(S > 1)>(ops, r, Y, lane);

    SegState ss;
    int n_closest = 0;   // closest-hit queries of this lane's ray so far
    WinRec rec;
    rec_start<true>(rec, op, vt, w);
    ss.alive = px.valid;
    ss.pending = op.ess && px.valid;
    ss.seg_i = 0;
    ss.a = tn;
    ss.cl_lo = tn;
    const float dS = op.dt * (float)NS;
    Window win;
    const float seg_max = (float)NS * (op.adaptive ? op.dt_max : op.dt);
    win.len_min = (float)NS * (op.adaptive ? op.dt_min : op.dt);
    win.len = (float)op.window_segments * seg_max;
    win.len_max = fmaxf(8.0f * seg_max, 2.0f * win.len);
    win.valid = false;
    win.hi = -kInf;
    win.count = 0;
    win.kind = SRC_LIST;
    win.chunked = false;
    win.t.paused = false;
    win.t.z1 = n_active;
    float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
    int32_t cnt[kNStatUsed];
#pragma unroll
    for (int k = 0; k < kNStatUsed; k++) cnt[k] = 0;
    cnt[ST_T_END] = __float_as_int(tf);
    // statistics builds also time the phases of the tile (shader clock)
    int64_t cyc_collect = 0, cyc_closest = 0, cyc_t0 = 0, cyc_tile = stats ? clock64() : 0;
    int64_t cyc_boxstat = 0;   // statistics-only work inside the collection
    float prev_a = -kInf, prev_b = -kInf;
    int n_dump = 0;

    for (;;) {
      if (stats) cyc_t0 = clock64();
      if (op.ess)
        closest_pass<S>(s, op, n_active, r, tn, tf, dS, ss, ls.error_flag,
                     stats ? &cnt[ST_CLOSEST] : nullptr, n_closest, px.ray);
      if (stats) cyc_closest += clock64() - cyc_t0;
      if (ss.alive) {
        const float a0 = grid ? fmaf((float)(ss.seg_i * NS), op.dt, tn) : ss.a;
        if (!(a0 < tf)) ss.alive = false;
        else if (!(T > op.t_eps)) {
          ss.alive = false;
          if (stats) cnt[ST_T_END] = __float_as_int(a0);
        }
      }
      if (ballot(ss.alive) == 0) break;
      float a = 0.0f, b = 0.0f, dt = op.dt;
      Samples sp;
      if (ss.alive) {
        if (!segment<NS>(op, grid, ss, tn, T, a, b, dt, sp)) {   // no progress in FP32
          ss.alive = false;
          if (ls.error_flag) *ls.error_flag = 4;
        }
      }
      if (!ss.alive) { sp.t0 = 0.0f; sp.dt = 0.0f; }
      bool go;
      if (stats) cyc_t0 = clock64();
      ensure_window<WIN_SEARCH>(s, op, M, r, lane, n_active, ss.alive, a, b, win, sm, ls.error_flag,
                    cnt[ST_NODES], cnt[ST_LEAVES], cnt[ST_WINDOWS], go, rec,
                    stats ? &cyc_boxstat : nullptr);
      if (stats) cyc_collect += clock64() - cyc_t0;
      if (stats && go && win.chunked) cnt[ST_CHUNKED]++;
      const float a_min = wave_min(go ? a : kInf), b_max = wave_max(go ? b : -kInf);
      const float lo = go ? a : kInf, hi = go ? b : -kInf;
      float sg[NL], W0[NL], W1[NL], W2[NL];
#pragma unroll
      for (int k = 0; k < NL; k++) { sg[k] = 0.0f; W0[k] = W1[k] = W2[k] = 0.0f; }
      int nhit = 0;

      do {
        for_each_candidate<CAND_MARK, (S > 1)>(win.kind, s, M, win.count, lane, a_min, b_max, n_active,
                                             r, ops, go, lo, hi, [&] { if (stats) cnt[ST_CAND]++; },
                                            [&](int, int j, const Cand &g, bool hit) {
        const Chord &c = g.ch;
        if (stats) cnt[ST_CAND_HIT]++;
        if (hit) {
          nhit++;
          if (stats && !(c.tin <= prev_b && c.tout >= prev_a)) cnt[ST_Q]++;
          if (DUMP) {
            if (n_dump < out.dump_cap) {
              out.dump_a[(size_t)dump_slot * out.dump_cap + n_dump] = a;
              out.dump_ids[(size_t)dump_slot * out.dump_cap + n_dump] = (int32_t)s.perm[j];
            }
            n_dump++;
          }
          const SampleExp se = sample_exp(g.k2, g.l2sig, c, sp);
          // samples no lane sees inside the Gaussian are skipped with a
          // uniform branch (their terms are exact zeros)
          if constexpr (S == 1) {
            // the colour record's loads go out before the sample weights,
            // which do not need them
            const ColRec rc = colour_load(s.col, j);
            float wk[NS];
            uint32_t live = 0;   // (uniform) samples some lane sees inside the Gaussian
#pragma unroll
            for (int k = 0; k < NS; k++) {
              const float x = se.at(k);
              const bool in = x >= se.e_min;
              wk[k] = 0.0f;
              if (ballot(in) != 0) {
                wk[k] = in ? __builtin_amdgcn_exp2f(x) : 0.0f;
                live |= 1u << k;
              }
            }
            float cr, cg, cb;
            colour_eval(rc, Y, cr, cg, cb);
            if constexpr (SG) sg_colour(s.sg, j, r.dx, r.dy, r.dz, cr, cg, cb);
#pragma unroll
            for (int k = 0; k < NS; k++) {
              if (!(live & (1u << k))) continue;
              sg[k] += wk[k];
              W0[k] = fmaf(wk[k], cr, W0[k]);
              W1[k] = fmaf(wk[k], cg, W1[k]);
              W2[k] = fmaf(wk[k], cb, W2[k]);
            }
          } else {
            float cr = g.cr, cg = g.cg, cb = g.cb;
            if constexpr (SG) sg_colour(s.sg, j, r.dx, r.dy, r.dz, cr, cg, cb);
#pragma unroll
            for (int k = 0; k < NL; k++) {
              const float x = se.at((float)(k * S) + (float)sub);
              const bool in = x >= se.e_min;
              if (ballot(in) == 0) continue;
              const float w = in ? __builtin_amdgcn_exp2f(x) : 0.0f;
              sg[k] += w;
              W0[k] = fmaf(w, cr, W0[k]);
              W1[k] = fmaf(w, cg, W1[k]);
              W2[k] = fmaf(w, cb, W2[k]);
            }
          }
        }
      }, [](int, int, uint32_t) {});
        // the entries this pass hit, for a replaying backward
        if (op.replay_mode == 1 && win.kind == SRC_LIST) rec_put_marks(rec, op, M, win.count, lane);
      } while ([&] {
        if (stats) cyc_t0 = clock64();
        const bool more = next_chunk<WIN_SEARCH>(s, op, M, r, lane, n_active, go, a, b, win, sm,
                                     ls.error_flag, cnt[ST_NODES], cnt[ST_LEAVES], cnt[ST_WINDOWS],
                                     rec, stats ? &cyc_boxstat : nullptr);
        if (stats) cyc_collect += clock64() - cyc_t0;
        return more;
      }());

      // an empty segment restarts at the next closest hit: inside the window
      // from the list, otherwise through a closest-hit traversal
      const bool empty = go && nhit == 0;
      float best = kInf;
      if (op.ess && win.kind == SRC_LIST && !win.chunked && ballot(empty)) {
        const float bmin = wave_min(empty ? b : kInf);
        for_each_candidate<CAND_ALL, false>(SRC_LIST, s, M, win.count, lane, bmin, kInf, n_active,
                                            r, ops, empty, b, win.hi, [] {},
                                            [&](int, int, const Cand &g, bool hit) {
          if (hit) best = fminf(best, fmaxf(g.ch.tin, b));
        }, [](int, int, uint32_t) {});
      }
      // the step's per-sample sums and restarts, for a replaying backward
      if (op.replay_mode == 1 && op.sample_rec)
        rec_put_samples<NL>(rec, op, go && nhit > 0, empty, best, sg, W0, W1, W2, lane);
      const bool shade = go && nhit > 0;
      if (stats && shade) { cnt[ST_SEGMENTS]++; cnt[ST_P] += nhit; }
      if (ballot(shade) != 0) {
#pragma unroll
        for (int k0 = 0; k0 < NL; k0++) {
          // samples k0 S .. k0 S + S - 1 of the ray, in order, in all its lanes
          float v[S], w0[S], w1[S], w2[S];
          ray_lanes<S>(sg[k0], v);
          ray_lanes<S>(W0[k0], w0);
          ray_lanes<S>(W1[k0], w1);
          ray_lanes<S>(W2[k0], w2);
#pragma unroll
          for (int i = 0; i < S; i++) {
            if (shade && sp.t(k0 * S + i) < tf) {
              if (stats) cnt[ST_SAMPLES]++;
              if (v[i] > 0.0f) {
                const float x = v[i] * dt;
                const float f = T * (one_minus_exp_neg(x) * __builtin_amdgcn_rcpf(v[i]));
                C0 = fmaf(f, w0[i], C0);
                C1 = fmaf(f, w1[i], C1);
                C2 = fmaf(f, w2[i], C2);
                T *= exp_neg(x);
              }
            }
          }
        }
      }
      if (go) {
        if (nhit > 0) {
          prev_a = a;
          prev_b = b;
        }
        step_after(op, grid, nhit > 0, best, tn, dS, b, ss);
      }
    }

    rec_finish(rec, op, lane);
    if (stats) {
      cnt[ST_BOX_ONLY] += sm->cnt_box[lane];
      cnt[ST_KCYC_COLLECT] = (int32_t)((cyc_collect - cyc_boxstat) >> 10);
      cnt[ST_KCYC_CLOSEST] = (int32_t)(cyc_closest >> 10);
      cnt[ST_KCYC_TILE] = (int32_t)((clock64() - cyc_tile - cyc_boxstat) >> 10);
    }
    if (DUMP) {
      if (px.valid) out.dump_count[dump_slot] = n_dump;
    } else if (px.valid && sub == 0) {
      out.rgb[3 * (size_t)px.ray + 0] = fmaf(T, op.bg[0], C0);
      out.rgb[3 * (size_t)px.ray + 1] = fmaf(T, op.bg[1], C1);
      out.rgb[3 * (size_t)px.ray + 2] = fmaf(T, op.bg[2], C2);
      out.T[px.ray] = T;
      if (stats) {
        for (int k = 0; k < kNStatUsed; k++) out.stats[(size_t)px.ray * kNStat + k] = cnt[k];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Lobe gradients of Gaussian j for one pass-B visit.  The lane's dL/dc is
// S G (S = sum_k w_k T_k phi_k, zero where the lane missed j), so per lobe
// with g = exp(lambda (u.d - 1)) and A = a.G:
//   dL/da = S g G,  dL/dlambda = S A g (u.d - 1),  h = S A g d,
// h being dL/du / lambda (the finalisation multiplies by lambda and takes
// the component across u).  Two lobes (16 slots) at a time are summed over
// the wave and added with one atomic per slot.
__device__ __forceinline__ void sg_slots(const float *sg, float *sgacc, int j, float S, float G0,
                                         float G1, float G2, const Ray &r, int lane) {
  cfloat4p p = as_const4(sg) + (size_t)(kSgFloats / 4) * j;
#pragma unroll 1
  for (int pair = 0; pair < (kMaxSg + 1) / 2; pair++) {
    float v[16];
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const int k = 2 * pair + h;
      float *o = v + 8 * h;
      if (k < kMaxSg) {
        const vf4 a = p[2 * k], u = p[2 * k + 1];
        const float cosang = fmaf(u.x, r.dx, fmaf(u.y, r.dy, u.z * r.dz));
        const float sgv = S * __builtin_amdgcn_exp2f(a.w * kLog2e * (cosang - 1.0f));
        const float sa = sgv * fmaf(a.x, G0, fmaf(a.y, G1, a.z * G2));
        o[0] = sgv * G0; o[1] = sgv * G1; o[2] = sgv * G2;
        o[3] = sa * (cosang - 1.0f);
        o[4] = sa * r.dx; o[5] = sa * r.dy; o[6] = sa * r.dz;
        o[7] = 0.0f;
      } else {
#pragma unroll
        for (int e = 0; e < 8; e++) o[e] = 0.0f;
      }
    }
    const float mine = wave_sum_slots16(v, lane);
    if ((lane & 3) == 0 && 16 * pair + (lane >> 2) < kMaxSg * kSgLobeFloats)
      unsafeAtomicAdd(sgacc + (size_t)kSgAccFloats * j + 16 * pair + (lane >> 2), mine);
  }
}

// ---------------------------------------------------------------------------
// Backward kernel: replays the forward's segments from the same window lists
// (or brute force) in the same order, takes each
// segment's per-sample sums from the forward's record (or sums them again
// where there is none), recomputes the transmittance before every sample,
// derives dL/dsigma_k and dL/dW_k, then revisits the Gaussians some lane hit
// for their parameter adjoints.  The 16
// geometry and density slots are summed over the wave (through LDS, or by DPP
// and half-wave swaps), four Gaussians' to one atomic instruction; the
// SH-coefficient slots, a per-ray
// constant times one scalar per (ray, Gaussian), are staged 16 Gaussians at a
// time and multiplied out on the matrix cores.

// REPLAY: every tile's record is complete, per-sample sums included; nothing
// there walks the tree or sums Gaussians again, and without that code the
// kernel fits two waves per SIMD without spills.  (Three, at 168 registers,
// spill into the candidate loop: 37.8 ms against 31.5.)  Otherwise the tiles
// are recorded or not, each for itself.  Whether every record found room is
// known on the device only, so both are launched and the waves of one leave
// at once (op.either).  With a replaying launch for the recorded tiles and one
// of this kind for the rest, each waited for its own slowest tiles: 100k
// Gaussians, 800x800, fixed step, 1490 tiles of 10000 unrecorded, 11.8 ms
// against 9.7; 1M, 4 x 1024x768, 22150 of 49152, 68.4 against 64.0; outdoor
// 3M, 1297x840, 2440 of 17115, 36.6 against 37.3.
template <int NS, int S, bool SG, bool REPLAY>
__global__ __launch_bounds__(kWave, 2) void k_backward(SceneDev s, ViewTable vt, MarchOpts op,
                                                    BwdIn in, LaunchShape ls) {
  constexpr int kMode = REPLAY ? WIN_REPLAY : WIN_BOTH;
  // Where a tile may have to search, with one lane a ray: colours only for the
  // groups some lane hits, and the slots summed in registers.  Half of a
  // list's candidates and nearly all of a brute-force pass are hit by no lane,
  // and sum_rows16's buffer beside the search's memory left seven waves to a
  // CU.  Backward ms before and after: 1M Gaussians, 4 x 1024x768, searching
  // everything 85.0 and 76.5, searches recorded 48.0 and 44.4; 1k, 640x480,
  // brute force 48.6 and 30.5; 100k, 800x800, fixed step, searches recorded 9.5
  // and 8.7.  (Vector colours of the hits alone: 84.8, 54.1, 30.0 and 10.3.)
  constexpr bool kLate = !REPLAY && S == 1, kRows = REPLAY && S == 1;
  __shared__ std::conditional_t<REPLAY, ListMem, WaveMem> M;
  __shared__ ShMem<kRows> sb;
  static_assert((sizeof(M) + sizeof(sb)) * kBwdWavesPerCu <= kLdsBytes, "resident waves");
  ShBatch shb;
  constexpr int kRays = 64 / S, NL = NS / S;   // rays of the tile; samples of a ray per lane
  const int lane = threadIdx.x;
  const int sub = lane / kRays;                // this lane's samples: sub, sub + S, ...
  const int n_active = uniform_int(s.counters[0]);
  const bool grid = !op.adaptive && op.ess != 2;
  if (!marches_any(s, op, vt)) return;
  if (op.either) {
    if (REPLAY != (op.wrec[kWrecFull] == 0u)) return;
  }
  bool first = true;
  for (;;) {
    int w;
    if (op.persistent) {
      w = pop_tile(ls.queue, vt.n_tiles, blockIdx.x & 7, lane);
      if (w < 0) break;
    } else {
      if (!first) break;
      w = xcd_block(blockIdx.x, gridDim.x);
      if (w >= vt.n_tiles) break;
    }
    first = false;

    const Pixel px = tile_pixel(vt, op, w, lane & (kRays - 1), kRays);
    const View &V = vt.v[px.view];
    if (!marches_view(s, op, V)) continue;
    WinRec rec;
    rec_start<false>(rec, op, vt, w);
    if (REPLAY && !rec.ok) {   // (cannot happen)
      if (ls.error_flag) *ls.error_flag = 5;
      continue;
    }
    const Ray r = make_ray(V, px.px, px.py);
    const float tn = V.t_near, tf = V.t_far;
    float Y[16];
    sh_basis(op.sh_k, r.dx, r.dy, r.dz, Y);
    float Gc0 = 0, Gc1 = 0, Gc2 = 0, GCf = 0;
    if (px.valid) {
      const size_t q = 3 * (size_t)px.ray;
      Gc0 = in.grad_rgb[q];
      Gc1 = in.grad_rgb[q + 1];
      Gc2 = in.grad_rgb[q + 2];
      const float gT = in.grad_T ? in.grad_T[px.ray] : 0.0f;
      // G . C_fin + g_T T_fin; the colour still to come behind sample k is
      // C_fin - (prefix through k), kept as the running scalar GP = G . prefix
      GCf = Gc0 * in.rgb[q] + Gc1 * in.rgb[q + 1] + Gc2 * in.rgb[q + 2] + gT * in.T[px.ray];
    }
    sh_batch_start(shb, sb, Y, Gc0, Gc1, Gc2, lane);
    TileOps<S> ops;
    tile_ops<true>(ops, r, Y, lane);
    float GP = 0.0f;
    SegState ss;
    int n_closest = 0;   // closest-hit queries of this lane's ray so far
    ss.alive = px.valid;
    ss.pending = op.ess && px.valid;
    ss.seg_i = 0;
    ss.a = tn;
    ss.cl_lo = tn;
    const float dS = op.dt * (float)NS;
    Window win;
    const float seg_max = (float)NS * (op.adaptive ? op.dt_max : op.dt);
    win.len_min = (float)NS * (op.adaptive ? op.dt_min : op.dt);
    win.len = (float)op.window_segments * seg_max;
    win.len_max = fmaxf(8.0f * seg_max, 2.0f * win.len);
    win.valid = false;
    win.hi = -kInf;
    win.count = 0;
    win.kind = SRC_LIST;
    win.chunked = false;
    win.t.paused = false;
    win.t.z1 = n_active;
    int32_t dummy_nodes = 0, dummy_leaves = 0, dummy_windows = 0;
    float T = 1.0f;

    for (;;) {
      if (op.ess) closest_pass<S>(s, op, n_active, r, tn, tf, dS, ss, ls.error_flag, nullptr, n_closest, px.ray);
      if (ss.alive) {
        const float a0 = grid ? fmaf((float)(ss.seg_i * NS), op.dt, tn) : ss.a;
        if (!(a0 < tf) || !(T > op.t_eps)) ss.alive = false;
      }
      if (ballot(ss.alive) == 0) break;
      float a = 0.0f, b = 0.0f, dt = op.dt;
      Samples sp;
      if (ss.alive) {
        if (!segment<NS>(op, grid, ss, tn, T, a, b, dt, sp)) {
          ss.alive = false;
          if (ls.error_flag) *ls.error_flag = 4;
        }
      }
      if (!ss.alive) { sp.t0 = 0.0f; sp.dt = 0.0f; }
      bool go;
      ensure_window<kMode>(s, op, M, r, lane, n_active, ss.alive, a, b, win, nullptr, ls.error_flag,
                    dummy_nodes, dummy_leaves, dummy_windows, go, rec);
      const float a_min = wave_min(go ? a : kInf), b_max = wave_max(go ? b : -kInf);
      const float lo = go ? a : kInf, hi = go ? b : -kInf;
      // only G . W_k enters the adjoints, so pass A sums the Gaussians'
      // weights times G . c_l, one scalar per sample
      float sg[NL], GW[NL];
#pragma unroll
      for (int k = 0; k < NL; k++) { sg[k] = 0.0f; GW[k] = 0.0f; }
      int nhit = 0;
      // a replayed tile reads the forward's per-sample sums from its record;
      // pass A then only moves through the step's lists and marks
      const bool from_rec = REPLAY || (op.replay_mode == 2 && rec.ok && op.sample_rec);

      // pass A: the forward's per-sample sums, in the forward's order
      do {
        const bool use_marks = rec_next_marks(rec, op, M, win.count, win.kind, lane, ls.error_flag);
        if constexpr (!REPLAY)
        if (!from_rec)
        for_each_candidate<CAND_MARK, true, kLate>(win.kind, s, M, win.count, lane, a_min, b_max, n_active,
                                            r, ops, go, lo, hi, [] {},
                                            [&](int, int j, const Cand &g, bool hit) {
        const Chord &c = g.ch;
        if (hit) {
          nhit++;
          float cr = g.cr, cg = g.cg, cb = g.cb;
          if constexpr (SG) sg_colour(s.sg, j, r.dx, r.dy, r.dz, cr, cg, cb);
          const float gc = fmaf(Gc0, cr, fmaf(Gc1, cg, Gc2 * cb));
          const SampleExp se = sample_exp(g.k2, g.l2sig, c, sp);
#pragma unroll
          for (int k = 0; k < NL; k++) {
            const float x = S == 1 ? se.at(k) : se.at((float)(k * S) + (float)sub);
            const float w = x >= se.e_min ? __builtin_amdgcn_exp2f(x) : 0.0f;
            sg[k] += w;
            GW[k] = fmaf(w, gc, GW[k]);
          }
        }
      }, [](int, int, uint32_t) {}, use_marks);
      } while (next_chunk<kMode>(s, op, M, r, lane, n_active, go, a, b, win, nullptr, ls.error_flag,
                            dummy_nodes, dummy_leaves, dummy_windows, rec));
      float best = kInf;
      if (from_rec)
        nhit = rec_get_samples<NL>(rec, op, go, Gc0, Gc1, Gc2, sg, GW, &best, lane, ls.error_flag) ? 1 : 0;

      // per-sample adjoints: dL/dsigma_k (into sg) and T_k phi_k (into GW);
      // dL/dW_k is G T_k phi_k
      const bool any = go && nhit > 0;
      if (ballot(any) != 0) {
#pragma unroll
        for (int k0 = 0; k0 < NL; k0++) {
          // samples k0 S .. k0 S + S - 1 of the ray, in order, in all its lanes
          float v[S], gw[S], own_sig = 0.0f, own_w = 0.0f;
          ray_lanes<S>(sg[k0], v);
          ray_lanes<S>(GW[k0], gw);
#pragma unroll
          for (int i = 0; i < S; i++) {
            float dsig = 0.0f, dW = 0.0f;
            if (any && sp.t(k0 * S + i) < tf && v[i] > 0.0f) {
              const float x = v[i] * dt;
              const float E = exp_neg(x);
              const float rs = __builtin_amdgcn_rcpf(v[i]);
              const float alpha = one_minus_exp_neg(x);
              const float phi = alpha * rs;
              // d(alpha/sigma)/dsigma = dt^2 f'(x), f(x) = (1 - e^-x)/x
              const float dphi = x < 1e-2f
                  ? dt * dt * (-0.5f + x * (1.0f / 3.0f - x * (0.125f - x * (1.0f / 30.0f))))
                  : (x * E - alpha) * rs * rs;
              GP = fmaf(T * phi, gw[i], GP);
              dsig = T * dphi * gw[i] - dt * (GCf - GP);
              dW = T * phi;
              T *= E;
            }
            if (S == 1 || sub == i) { own_sig = dsig; own_w = dW; }
          }
          sg[k0] = own_sig;
          GW[k0] = own_w;
        }
      }

      // pass B: per-Gaussian adjoints
      if (ballot(any) != 0) {
        float red[4] = {0.0f, 0.0f, 0.0f, 0.0f};   // the group's reduced slots, one candidate each
        auto pass_b = [&](int ci, int j, const Cand &g, bool hit) {
          const Chord &c = g.ch;
          float sw = 0.0f;   // sum over the lane's samples of w_k T_k phi_k
          float v[16];
#pragma unroll
          for (int e2 = 0; e2 < 16; e2++) v[e2] = 0.0f;
          if (hit) {
            float cr = g.cr, cg = g.cg, cb = g.cb;
            if constexpr (SG) sg_colour(s.sg, j, r.dx, r.dy, r.dz, cr, cg, cb);
            const float gc = fmaf(Gc0, cr, fmaf(Gc1, cg, Gc2 * cb));
            const SampleExp se = sample_exp(g.k2, g.l2sig, c, sp);
            // dL/dw_k = dsigma_k + G.c_l T_k phi_k; dq_k = -w_k dL/dw_k / 2
            // moments over u_k = u_0 + k dt from sums over the sample index
            float ds = 0.0f, F1 = 0.0f, F2 = 0.0f;
            // four samples at a time, skipped when no lane sees one of them
            // inside the Gaussian: their terms are zeros (1M Gaussians, 2.5 of 8
            // samples are seen: 30.5 -> 29.95 ms; a test for each sample costs
            // what it saves, 30.6 ms).  Lanes sharing a ray hold few samples
            // and take them all.
            constexpr int kSkip = NL < 4 ? NL : 4;
#pragma unroll
            for (int k0 = 0; k0 < NL; k0 += kSkip) {
              float x[kSkip], top = -kInf;
#pragma unroll
              for (int q = 0; q < kSkip; q++) {
                x[q] = S == 1 ? se.at(k0 + q) : se.at((float)((k0 + q) * S) + (float)sub);
                top = fmaxf(top, x[q]);
              }
              if (S == 1 && ballot(top >= se.e_min) == 0) continue;
#pragma unroll
              for (int q = 0; q < kSkip; q++) {
                const int k = k0 + q;
                const float kf = S == 1 ? (float)k : (float)(k * S) + (float)sub;
                const float e = __builtin_amdgcn_exp2f(x[q]);
                const float w = x[q] >= se.e_min ? e : 0.0f;
                const float wdw = w * fmaf(GW[k], gc, sg[k]);
                ds += wdw;
                F1 = fmaf(kf, wdw, F1);
                F2 = fmaf(kf * kf, wdw, F2);
                sw = fmaf(w, GW[k], sw);
              }
            }
            const float u0 = sp.t0 - c.ts;
            const float E1 = fmaf(u0, ds, sp.dt * F1);                         // sum wdw u
            const float E2 = fmaf(u0, fmaf(u0, ds, 2.0f * sp.dt * F1), sp.dt * sp.dt * F2);
            const float D0 = -0.5f * ds, D1 = -0.5f * E1, D2 = -0.5f * E2;
            // z_k = p + u_k d' with p = o' + t* d' (closest approach, local
            // frame), and the closest-approach point's world offset P from
            // the mean
            const float px = fmaf(c.ts, g.dx, g.ox), py = fmaf(c.ts, g.dy, g.oy),
                        pz = fmaf(c.ts, g.dz, g.oz);
            const float Ps[3] = {fmaf(c.ts, r.dx, g.ex), fmaf(c.ts, r.dy, g.ey),
                                 fmaf(c.ts, r.dz, g.ez)};
            const float Zs[3] = {fmaf(D0, px, D1 * g.dx), fmaf(D0, py, D1 * g.dy),
                                 fmaf(D0, pz, D1 * g.dz)};
            const float Us[3] = {fmaf(D1, px, D2 * g.dx), fmaf(D1, py, D2 * g.dy),
                                 fmaf(D1, pz, D2 * g.dz)};
            const float dd[3] = {r.dx, r.dy, r.dz};
            v[0] = Zs[0]; v[1] = Zs[1]; v[2] = Zs[2];
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
              for (int jj = 0; jj < 3; jj++) v[3 + 3 * i + jj] = fmaf(Zs[i], Ps[jj], Us[i] * dd[jj]);
            v[12] = fmaf(D0, px * px, fmaf(2.0f * D1, px * g.dx, D2 * g.dx * g.dx));
            v[13] = fmaf(D0, py * py, fmaf(2.0f * D1, py * g.dy, D2 * g.dy * g.dy));
            v[14] = fmaf(D0, pz * pz, fmaf(2.0f * D1, pz * g.dz, D2 * g.dz * g.dz));
            v[15] = ds;
          }
          // the geometry and density slots are summed over the wave; the SH
          // slots go through the matrix-core batch
          sb.s[shb.n * kSbStride + lane] = sw;
          shb.id = lane == shb.n ? j : shb.id;
          shb.n++;
          // (through LDS the waves of a full chip gain 0.8 ms in 31.2, 1M
          // Gaussians, 4 x 1024x768; a launch of few waves waits for it: 22.8 ms
          // against 20.8, 100k, 8 x 160x121 one by one)
          if constexpr (kRows) {
            red[ci] = sum_rows16(sb.r, v, lane);
          } else {
            float t[16];
#pragma unroll
            for (int e2 = 0; e2 < 16; e2++) t[e2] = v[4 * (e2 & 3) + (e2 >> 2)];
            red[ci] = wave_sum_slots16(t, lane);
          }
          if constexpr (SG) sg_slots(s.sg, in.sgacc, j, hit ? sw : 0.0f, Gc0, Gc1, Gc2, r, lane);
        };
        // a group's atomics go out as one instruction, behind the next group's
        // loads: 16 consecutive floats (one 64-byte line) of each of the four
        // Gaussians, slot lane & 15 of candidate lane >> 4
        auto put_b = [&](int ids, int first, uint32_t hits) {
          if (hits != 0) {
            float mine;
            if constexpr (kRows) {
              // red[c]: slot lane & 15 summed over one row of lanes
              mine = swap16_sum(swap32_sum(red[0], red[2]), swap32_sum(red[1], red[3]));
            } else {
              // red[c]: sum lane >> 2, which is slot 4 (i & 3) + (i >> 2)
              transpose_rows(red);
              const float even = (lane & 2) ? red[2] : red[0], odd = (lane & 2) ? red[3] : red[1];
              mine = (lane & 1) ? odd : even;
            }
            const uint32_t j = (uint32_t)__shfl(ids, first + (lane >> 4), 64);
            float *dst = in.acc + (size_t)kAccFloats * j + (lane & 15);
            // (the densification statistic needs each view's mean slots apart)
            if (in.zview && (lane & 15) < 3)
              dst = in.zview + ((size_t)px.view * s.n + j) * 3 + (lane & 15);
            if ((hits >> (lane >> 4)) & 1u) unsafeAtomicAdd(dst, mine);
          }
          if (shb.n > 12) sh_batch_flush(shb, sb, in.acc, op.sh_k, lane);
        };
        // the list still holds the whole window, or the segment's last Z
        // chunk [zlast, end), its entries marked by pass A; a chunked segment
        // then visits [0, zlast): re-read from the record with the forward's
        // marks when replaying, else collected again
        const int zlast = win.chunked ? win.t.z0 : 0;
        const bool earlier = win.chunked && zlast > 0;
        const bool reread = earlier && rec.ok;
        uint32_t off = win.rec_first;
        int n_cur = win.count, kind_cur = win.kind;
        bool marked = true;      // visit the marked entries only
        for (bool cur = true;; cur = false) {
          if (!cur) {
            if (!earlier) break;
            if (reread) {
              if (off == win.rec_last || off == kWrecNone) break;
              uint32_t next, after;
              const int c = rec_load(op, M, off, lane, &next);
              n_cur = c > 0 ? c : 0;
              if (c < 0 || next == kWrecNone || !rec_load_marks(op, M, next, n_cur, lane, &after)) {
                if (ls.error_flag) *ls.error_flag = 5;
                break;
              }
              off = after;
            } else if constexpr (REPLAY) {
              break;
            } else {
              if (marked)
                first_chunk(s, M, r, lane, n_active, any, a, b, zlast, win, nullptr, ls.error_flag,
                            dummy_nodes, dummy_leaves, dummy_windows);
              else if (!next_chunk<kMode>(s, op, M, r, lane, n_active, any, a, b, win, nullptr,
                                         ls.error_flag, dummy_nodes, dummy_leaves, dummy_windows, rec))
                break;
              marked = false;
              n_cur = win.count;
            }
            kind_cur = SRC_LIST;
          }
          for_each_candidate<CAND_FILTER, true, kLate>(kind_cur, s, M, n_cur, lane, a_min, b_max, n_active,
                                                r, ops, any, lo, hi, [] {}, pass_b, put_b, marked);
        }
      }

      // restart after an empty segment: from the list inside the window, else
      // through the closest-hit traversal (same decisions as the forward)
      const bool empty = go && nhit == 0;
      if constexpr (!REPLAY)
      if (!from_rec && op.ess && win.kind == SRC_LIST && !win.chunked && ballot(empty)) {
        const float bmin = wave_min(empty ? b : kInf);
        for_each_candidate<CAND_ALL, false>(SRC_LIST, s, M, win.count, lane, bmin, kInf, n_active,
                                            r, ops, empty, b, win.hi, [] {},
                                            [&](int, int, const Cand &g, bool hit) {
          if (hit) best = fminf(best, fmaxf(g.ch.tin, b));
        }, [](int, int, uint32_t) {});
      }
      if (go) step_after(op, grid, nhit > 0, best, tn, dS, b, ss);
    }
    sh_batch_flush(shb, sb, in.acc, op.sh_k, lane);
  }
}

// ---------------------------------------------------------------------------
// Gradient finalisation: chain rule from the per-Gaussian accumulators to the
// user parameters (means, log-scales, quaternions through normalisation,
// density, SH), scattered to user order.  Bound by memory: 300 bytes read and
// 236 written a Gaussian.  A block takes its 256 Gaussians' SH rows element by
// element -- consecutive threads write consecutive floats of a user row -- and
// then one Gaussian a thread for the rest (a thread a whole Gaussian, whose
// stores go to 64 rows at once, and clearing what it read: 0.78 ms at 1M
// against 0.30 ms and 0.04 ms for the backward's clear).
template <int SHK>
__global__ __launch_bounds__(256) void k_finalize(int64_t n, const int32_t *__restrict__ counters,
                                                  const uint32_t *__restrict__ perm,
                                                  const float *__restrict__ geom,
                                                  const float *__restrict__ acc,
                                                  const float *__restrict__ aux,
                                                  float *__restrict__ gm, float *__restrict__ gl,
                                                  float *__restrict__ gq, float *__restrict__ gd,
                                                  float *__restrict__ gsh, int accumulate) {
  constexpr int kRow = 3 * SHK;
  __shared__ uint32_t user[256];
  const int64_t i0 = (int64_t)blockIdx.x * 256;
  const int64_t i = i0 + threadIdx.x;
  const int n_here = (int)(n - i0 < 256 ? n - i0 : 256), n_act = counters[0];
  // overwrite mode never reads the output buffers (they may hold anything)
  auto put = [accumulate](float &dst, float v) { dst = accumulate ? dst + v : v; };
  if ((int)threadIdx.x < n_here) user[threadIdx.x] = perm[i];
  __syncthreads();
  for (int e = threadIdx.x; e < n_here * kRow; e += 256) {
    const int j = e / kRow, f = e - j * kRow, m = f / 3, ch = f - 3 * m;
    const float v = i0 + j < n_act ? acc[(size_t)kAccFloats * (i0 + j) + 16 + 16 * ch + m] : 0.0f;
    put(gsh[(size_t)kRow * user[j] + f], v);
  }
  if (i >= n) return;
  const int64_t u = user[threadIdx.x];
  if (i >= n_act) {   // inactive Gaussian: zero gradient
    for (int k = 0; k < 3; k++) { put(gm[3 * u + k], 0.0f); put(gl[3 * u + k], 0.0f); }
    for (int k = 0; k < 4; k++) put(gq[4 * u + k], 0.0f);
    put(gd[u], 0.0f);
    return;
  }
  float A[16];
  const float4 *accp = reinterpret_cast<const float4 *>(acc + (size_t)kAccFloats * i);
  for (int k = 0; k < 4; k++) {
    const float4 v = accp[k];
    A[4 * k] = v.x; A[4 * k + 1] = v.y; A[4 * k + 2] = v.z; A[4 * k + 3] = v.w;
  }
  const float *G = geom + (size_t)kGeomFloats * i;
  float Z[3] = {A[0], A[1], A[2]};
  // dL/dmu = -2 M^T Z
  for (int jj = 0; jj < 3; jj++)
    put(gm[3 * u + jj], -2.0f * (G[G_M + jj] * Z[0] + G[G_M + 3 + jj] * Z[1] + G[G_M + 6 + jj] * Z[2]));
  // dL/dl_i = -2 sum z_i^2 dq
  for (int k = 0; k < 3; k++) put(gl[3 * u + k], -2.0f * A[12 + k]);
  // dL/dR_ji = 2 G'_ij / s_i
  const float *X = aux + (size_t)kAuxFloats * i;
  float dR[9];
  for (int ii = 0; ii < 3; ii++)
    for (int jj = 0; jj < 3; jj++) dR[3 * jj + ii] = 2.0f * A[3 + 3 * ii + jj] / X[ii];
  const float w = X[3], x = X[4], y = X[5], z = X[6], qn = X[7];
  float dq[4];
  dq[0] = 2.0f * (-z * dR[1] + y * dR[2] + z * dR[3] - x * dR[5] - y * dR[6] + x * dR[7]);
  dq[1] = 2.0f * (y * dR[1] + z * dR[2] + y * dR[3] - 2.0f * x * dR[4] - w * dR[5] + z * dR[6] +
                  w * dR[7] - 2.0f * x * dR[8]);
  dq[2] = 2.0f * (-2.0f * y * dR[0] + x * dR[1] + w * dR[2] + x * dR[3] + z * dR[5] - w * dR[6] +
                  z * dR[7] - 2.0f * y * dR[8]);
  dq[3] = 2.0f * (-2.0f * z * dR[0] - w * dR[1] + x * dR[2] + w * dR[3] - 2.0f * z * dR[4] +
                  y * dR[5] + x * dR[6] + y * dR[7]);
  const float pr = dq[0] * w + dq[1] * x + dq[2] * y + dq[3] * z;
  const float qh[4] = {w, x, y, z};
  for (int k = 0; k < 4; k++) put(gq[4 * u + k], (dq[k] - pr * qh[k]) / qn);
  put(gd[u], A[15] / G[G_SIG]);
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = i; k < n; k += stride) p[k] = v;
}

// ---------------------------------------------------------------------------

// The kernels for tiles of 64 / split rays.  Statistics, hit dumps and the
// shortest segments run at split 1 only (set by the host).
template <int NS, bool SG>
static hipError_t fwd_dispatch(const SceneDev &s, const ViewTable &vt, const MarchOpts &op,
                               const FwdOut &out, const LaunchShape &ls, hipStream_t st) {
  if (op.split == 1) {
    // (the hit dump does not depend on colour and takes the plain kernel)
    if (out.dump_pix) k_forward<NS, 1, true, false><<<ls.grid, kWave, 0, st>>>(s, vt, op, out, ls);
    else if (out.stats) k_forward<NS, 1, false, true, SG><<<ls.grid, kWave, 0, st>>>(s, vt, op, out, ls);
    else k_forward<NS, 1, false, false, SG><<<ls.grid, kWave, 0, st>>>(s, vt, op, out, ls);
    return hipGetLastError();
  }
  if constexpr (NS >= 4) {
    if (out.dump_pix || out.stats) return hipErrorInvalidValue;
    if (op.split == 2) k_forward<NS, 2, false, false, SG><<<ls.grid, kWave, 0, st>>>(s, vt, op, out, ls);
    else if (op.split == 4) k_forward<NS, 4, false, false, SG><<<ls.grid, kWave, 0, st>>>(s, vt, op, out, ls);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <int NS, bool SG, bool REPLAY>
static hipError_t bwd_dispatch(const SceneDev &s, const ViewTable &vt, const MarchOpts &op,
                               const BwdIn &in, const LaunchShape &ls, hipStream_t st) {
  if (op.split == 1) {
    k_backward<NS, 1, SG, REPLAY><<<ls.grid, kWave, 0, st>>>(s, vt, op, in, ls);
    return hipGetLastError();
  }
  if constexpr (NS >= 4) {
    if (op.split == 2) k_backward<NS, 2, SG, REPLAY><<<ls.grid, kWave, 0, st>>>(s, vt, op, in, ls);
    else if (op.split == 4) k_backward<NS, 4, SG, REPLAY><<<ls.grid, kWave, 0, st>>>(s, vt, op, in, ls);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  return hipErrorInvalidValue;
}

template <bool REPLAY>
static hipError_t bwd_launch(const SceneDev &s, const ViewTable &vt, const MarchOpts &op,
                             const BwdIn &in, const LaunchShape &ls, hipStream_t st) {
  if (op.persistent) {
    hipError_t e = launch_fill(ls.queue, 8, 0u, st);
    if (e != hipSuccess) return e;
  }
  if (s.n_sg > 0)
    return op.n_s == 8 ? bwd_dispatch<8, true, REPLAY>(s, vt, op, in, ls, st) : hipErrorInvalidValue;
  switch (op.n_s) {
    case 1: return bwd_dispatch<1, false, REPLAY>(s, vt, op, in, ls, st);
    case 2: return bwd_dispatch<2, false, REPLAY>(s, vt, op, in, ls, st);
    case 4: return bwd_dispatch<4, false, REPLAY>(s, vt, op, in, ls, st);
    case 8: return bwd_dispatch<8, false, REPLAY>(s, vt, op, in, ls, st);
    case 16: return bwd_dispatch<16, false, REPLAY>(s, vt, op, in, ls, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_forward(const SceneDev &s, const ViewTable &vt, const MarchOpts &op,
                          const FwdOut &out, const LaunchShape &ls, hipStream_t st) {
  if (op.persistent) {
    hipError_t e = launch_fill(ls.queue, 8, 0u, st);
    if (e != hipSuccess) return e;
  }
  if (s.n_sg > 0)   // lobed colour (spherical Gaussians): N_s = 8 only (checked by the host)
    return op.n_s == 8 ? fwd_dispatch<8, true>(s, vt, op, out, ls, st) : hipErrorInvalidValue;
  switch (op.n_s) {
    case 1: return fwd_dispatch<1, false>(s, vt, op, out, ls, st);
    case 2: return fwd_dispatch<2, false>(s, vt, op, out, ls, st);
    case 4: return fwd_dispatch<4, false>(s, vt, op, out, ls, st);
    case 8: return fwd_dispatch<8, false>(s, vt, op, out, ls, st);
    case 16: return fwd_dispatch<16, false>(s, vt, op, out, ls, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_backward(const SceneDev &s, const ViewTable &vt, const MarchOpts &op,
                           const BwdIn &in, const LaunchShape &ls, hipStream_t st) {
  MarchOpts o = op;
  o.either = op.replay_mode == 2 && op.sample_rec;
  if (o.either) {
    const hipError_t e = bwd_launch<true>(s, vt, o, in, ls, st);
    if (e != hipSuccess) return e;
  }
  return bwd_launch<false>(s, vt, o, in, ls, st);
}

hipError_t launch_finalize_grads(const SceneDev &s, int sh_k, float *acc, float *g_means,
                                 float *g_log_scales, float *g_quats, float *g_density,
                                 float *g_sh, int accumulate, hipStream_t st) {
  const unsigned nb = (unsigned)((s.n + 255) / 256);
  auto k = sh_k == 1 ? k_finalize<1> : sh_k == 4 ? k_finalize<4> : sh_k == 9 ? k_finalize<9> : k_finalize<16>;
  k<<<nb, 256, 0, st>>>(s.n, s.counters, s.perm, s.geom, acc, s.aux, g_means, g_log_scales, g_quats,
                        g_density, g_sh, accumulate);
  return hipGetLastError();
}

// Lobe gradients to user order: per lobe, dL/da and dL/dlambda as summed;
// the axis through u = xi / |xi|: dL/dxi = lambda (h - (h.u) u) / |xi|.
// Absent lobes and inactive Gaussians get zeros.
__global__ __launch_bounds__(256) void k_finalize_sg(int64_t n, const int32_t *__restrict__ counters,
                                                     const uint32_t *__restrict__ perm,
                                                     const float *__restrict__ sg,
                                                     const float *__restrict__ sgacc, int n_sg,
                                                     float *__restrict__ g_sg, int accumulate) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t u = perm[i];
  const bool active = i < counters[0];
  for (int k = 0; k < n_sg; k++) {
    float out[kSgUserFloats] = {0, 0, 0, 0, 0, 0, 0};
    if (active) {
      const float *A = sgacc + (size_t)kSgAccFloats * i + kSgLobeFloats * k;
      const float *L = sg + (size_t)kSgFloats * i + kSgLobeFloats * k;
      if (L[7] > 0.0f) {
        const float h[3] = {A[4], A[5], A[6]};
        const float hu = h[0] * L[4] + h[1] * L[5] + h[2] * L[6];
        const float f = L[3] / L[7];
        out[0] = A[0]; out[1] = A[1]; out[2] = A[2];
        for (int e = 0; e < 3; e++) out[3 + e] = f * (h[e] - hu * L[4 + e]);
        out[6] = A[3];
      }
    }
    float *dst = g_sg + ((size_t)u * n_sg + k) * kSgUserFloats;
    for (int e = 0; e < kSgUserFloats; e++) dst[e] = accumulate ? dst[e] + out[e] : out[e];
  }
}

hipError_t launch_finalize_sg(const SceneDev &s, float *sgacc, float *g_sg, int accumulate,
                              hipStream_t st) {
  const unsigned nb = (unsigned)((s.n + 255) / 256);
  k_finalize_sg<<<nb, 256, 0, st>>>(s.n, s.counters, s.perm, s.sg, sgacc, s.n_sg, g_sg, accumulate);
  return hipGetLastError();
}

// Densification statistic of a batch of views (Sec. 3.5, Eq. 12).  The views'
// backward left each one's mean sums in zview [views][n][3]; a view's mean
// gradient is -2 M^T Z.  densify[user i] += |mu - o_v| / f_v * |grad_v|, views
// += grad_v != 0, view by view, and the sums go into the mean slots for the
// chain rule.  One launch marches the whole batch: view by view, a view of 320
// tiles lasted as long as its slowest tile (100k Gaussians, 8 x 160x121: 20.8
// ms backward against 4.0 ms).
__global__ __launch_bounds__(256) void k_densify(int64_t n, const int32_t *__restrict__ counters,
                                                 const uint32_t *__restrict__ perm,
                                                 const float *__restrict__ geom,
                                                 float *__restrict__ acc,
                                                 const float *__restrict__ zview, ViewTable vt,
                                                 float *__restrict__ densify,
                                                 int32_t *__restrict__ views) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n || i >= counters[0]) return;
  const float *G = geom + (size_t)kGeomFloats * i;
  float sum[3];
  for (int r = 0; r < 3; r++) sum[r] = acc[(size_t)kAccFloats * i + r];
  const uint32_t u = perm[i];
  float stat = densify[u];
  int32_t seen = 0;
  for (int v = 0; v < vt.n_views; v++) {
    const float *z = zview + ((size_t)v * n + i) * 3;
    for (int r = 0; r < 3; r++) sum[r] += z[r];
    float g2 = 0.0f;
    for (int c = 0; c < 3; c++) {
      const float gc = -2.0f * (G[G_M + c] * z[0] + G[G_M + 3 + c] * z[1] + G[G_M + 6 + c] * z[2]);
      g2 = fmaf(gc, gc, g2);
    }
    if (g2 > 0.0f) {
      const View &V = vt.v[v];
      const float ex = G[G_MU] - V.c2w[3], ey = G[G_MU + 1] - V.c2w[7], ez = G[G_MU + 2] - V.c2w[11];
      const float alpha = sqrtf(ex * ex + ey * ey + ez * ez) * (1.0f / V.fx);
      stat += alpha * sqrtf(g2);
      seen++;
    }
  }
  for (int r = 0; r < 3; r++) acc[(size_t)kAccFloats * i + r] = sum[r];
  if (seen) {
    densify[u] = stat;
    views[u] += seen;
  }
}

hipError_t launch_densify(const SceneDev &s, float *acc, const float *zview, const ViewTable &vt,
                          float *densify, int32_t *views, hipStream_t st) {
  const unsigned nb = (unsigned)((s.n + 255) / 256);
  k_densify<<<nb, 256, 0, st>>>(s.n, s.counters, s.perm, s.geom, acc, zview, vt, densify, views);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Statistics totals of one forward (int64, RGX_TOT_* order of the public
// header): per-block column sums of the per-ray counters, one atomic per
// column per block; the inactive Gaussians and the unrecorded tiles of the
// record are counted by the same launch.
enum { TOT_RAYS = 0, TOT_Q, TOT_P, TOT_SAMPLES, TOT_SEGMENTS, TOT_CLOSEST, TOT_NODES,
       TOT_BOX_ONLY, TOT_CHUNKED, TOT_INACTIVE, TOT_UNRECORDED, kNTot };

__global__ __launch_bounds__(256) void k_stat_totals(const int32_t *__restrict__ stats, int64_t rays,
                                                     int64_t n, const int32_t *__restrict__ counters,
                                                     const uint32_t *__restrict__ wrec_tile,
                                                     int64_t tiles, unsigned long long *totals) {
  constexpr int kCols = 8;
  const int cols[kCols] = {-1, ST_Q, ST_P, ST_SAMPLES, ST_SEGMENTS, ST_CLOSEST, ST_NODES, ST_BOX_ONLY};
  __shared__ unsigned long long red[kCols + 2][256];
  unsigned long long acc[kCols + 2];
#pragma unroll
  for (int c = 0; c < kCols + 2; c++) acc[c] = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < rays; r += stride) {
    const int32_t *row = stats + (size_t)r * kNStat;
    acc[0] += 1;
#pragma unroll
    for (int c = 1; c < kCols; c++) acc[c] += (unsigned long long)(uint32_t)row[cols[c]];
    acc[kCols] += (unsigned long long)(uint32_t)row[ST_CHUNKED];
  }
  if (wrec_tile)
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < tiles; t += stride)
      acc[kCols + 1] += wrec_tile[2 * t] == 1u ? 0ull : 1ull;
#pragma unroll
  for (int c = 0; c < kCols + 2; c++) red[c][threadIdx.x] = acc[c];
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h)
#pragma unroll
      for (int c = 0; c < kCols + 2; c++) red[c][threadIdx.x] += red[c][threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
#pragma unroll
    for (int c = 0; c < kCols; c++) atomicAdd(&totals[c], red[c][0]);
    atomicAdd(&totals[TOT_CHUNKED], red[kCols][0]);
    atomicAdd(&totals[TOT_UNRECORDED], red[kCols + 1][0]);
    if (blockIdx.x == 0) atomicAdd(&totals[TOT_INACTIVE], (unsigned long long)(n - counters[0]));
  }
}

hipError_t launch_stat_totals(const int32_t *stats, int64_t rays, const SceneDev &s,
                              const uint32_t *wrec_tile, int64_t tiles, int64_t *totals,
                              hipStream_t st) {
  hipError_t e = launch_fill(totals, 2 * kNTot, 0u, st);
  if (e != hipSuccess) return e;
  const int64_t work = rays > tiles ? rays : tiles;
  int64_t nb = (work + 255) / 256;
  if (nb > 2048) nb = 2048;
  if (nb < 1) nb = 1;
  k_stat_totals<<<(unsigned)nb, 256, 0, st>>>(stats, rays, s.n, s.counters, wrec_tile, tiles,
                                              reinterpret_cast<unsigned long long *>(totals));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Whole-ray AABB false positives (Sec. 3.4, Eq. 6; minimal AABB of Supp. B)
// of listed pixels of one view: Gaussians whose minimal AABB mu +/- L,
// L_a = k sqrt(sum_m R_am^2 s_m^2), meets the ray over [t_n, t_end] while the
// ellipsoid's chord does not.  One thread per ray walks the binary LBVH with
// its own stack.  The node boxes are padded unions of padded leaf boxes, so
// they contain every minimal AABB below them and the walk misses none; the
// leaves then take the exact (unpadded) test.  Internal nodes lie at most 86
// levels deep (the Karras split positions grow strictly down the tree over
// the 63-bit key extended by a 23-bit index), and the walk pushes one child
// per level, so 96 stack entries always suffice.
constexpr int kFpStack = 96;

__global__ __launch_bounds__(256) void k_false_positives(SceneDev s, View V, const int32_t *__restrict__ pix,
                                                         int n_rays, const float *__restrict__ t_end,
                                                         int32_t *__restrict__ count,
                                                         int32_t *__restrict__ err) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_rays) return;
  const int n_active = s.counters[0];
  const int p = pix[i];
  const Ray r = make_ray(V, p % V.width, p / V.width);
  const float lo = V.t_near, hi = t_end[i];
  int fp = 0;
  auto leaf = [&](int j) {
    const Gauss g = with_origin(load_gauss_lane(s.geom, j), r.ox, r.oy, r.oz);
    const float *X = s.aux + (size_t)kAuxFloats * j;
    const float sx = X[0], sy = X[1], sz = X[2];
    const float w = X[3], x = X[4], y = X[5], z = X[6];
    // rows of R(q) for the unit quaternion (w, x, y, z)
    const float R[9] = {1.0f - 2.0f * (y * y + z * z), 2.0f * (x * y - w * z), 2.0f * (x * z + w * y),
                        2.0f * (x * y + w * z), 1.0f - 2.0f * (x * x + z * z), 2.0f * (y * z - w * x),
                        2.0f * (x * z - w * y), 2.0f * (y * z + w * x), 1.0f - 2.0f * (x * x + y * y)};
    const float k = sqrtf(g.k2);
    const float mu[3] = {g.mx, g.my, g.mz}, o[3] = {r.ox, r.oy, r.oz}, d[3] = {r.dx, r.dy, r.dz};
    float enter = lo, leave = hi;
#pragma unroll
    for (int a = 0; a < 3; a++) {
      const float e2 = R[3 * a] * R[3 * a] * sx * sx + R[3 * a + 1] * R[3 * a + 1] * sy * sy +
                       R[3 * a + 2] * R[3 * a + 2] * sz * sz;
      const float L = k * sqrtf(e2);
      const float ta = (mu[a] - L - o[a]) / d[a], tb = (mu[a] + L - o[a]) / d[a];
      enter = fmaxf(enter, fminf(ta, tb));
      leave = fminf(leave, fmaxf(ta, tb));
    }
    const Chord c = chord(g, r);
    const bool ell = c.exists && c.tin <= hi && c.tout >= lo;
    if (enter <= leave && !ell) fp++;
  };
  if (n_active == 1) {
    leaf(0);
  } else if (n_active > 1) {
    int stack[kFpStack];
    int sp = 0, node = 0;
    for (;;) {
      const vf4 *np = reinterpret_cast<const vf4 *>(s.nodes) + 4 * node;
      const vf4 a = np[0], b = np[1], c = np[2], d = np[3];
      const int cl = __float_as_int(a.w), cr = __float_as_int(b.w);
      const bool hL = cl != kNoChild && box_hit(a.x, a.y, a.z, b.x, b.y, b.z, r, lo, hi);
      const bool hR = cr != kNoChild && box_hit(c.x, c.y, c.z, d.x, d.y, d.z, r, lo, hi);
      int next = -1;
      if (hL) {
        if (cl < 0) leaf(~cl); else next = cl;
      }
      if (hR) {
        if (cr < 0) leaf(~cr);
        else if (next < 0) next = cr;
        else if (sp < kFpStack) stack[sp++] = cr;
        else { if (err) *err = 6; fp = -1; break; }
      }
      if (next >= 0) { node = next; continue; }
      if (sp == 0) break;
      node = stack[--sp];
    }
  }
  count[i] = fp;
}

hipError_t launch_false_positives(const SceneDev &s, const View &v, const int32_t *pix, int32_t n_rays,
                                  const float *t_end, int32_t *count, int32_t *error_flag,
                                  hipStream_t st) {
  if (n_rays <= 0) return hipSuccess;
  k_false_positives<<<(unsigned)((n_rays + 255) / 256), 256, 0, st>>>(s, v, pix, n_rays, t_end, count,
                                                                      error_flag);
  return hipGetLastError();
}

hipError_t launch_fill(void *p, int64_t n_words, uint32_t value, hipStream_t st) {
  if (n_words <= 0) return hipSuccess;
  int64_t blocks = (n_words + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  k_fill_u32<<<(unsigned)blocks, 256, 0, st>>>((uint32_t *)p, n_words, value);
  return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t st) {
  return launch_fill(p, n, __builtin_bit_cast(uint32_t, v), st);
}

}  // namespace rgx
