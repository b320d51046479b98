// gfx950 kernels of the differentiable tile-based Gaussian-splatting rasterizer.
//
//   K1 k_project        per Gaussian, loop over views: Eq. 2, 4, 5 (+ low-pass), conic of
//                       the 2D splat (Eq. 3), SH colour, frustum cull, tile rectangle, tile count,
//                       block sums of the tile counts and of the visible records
//   K2 k_scan_pairs     exclusive scans of those block sums (one block, or of many by tiles)
//   K3/K4               the stable sort of the (tile id << 32 | depth bits) keys, without
//                       materialising them: k_compact + k_radix_* sort the visible records by
//                       depth bits (stable LSD, 8-bit digits: histogram / row scan /
//                       ballot-multisplit scatter; few: k_sort_small); k_bin_* then bin that depth order stably,
//                       first into tile rows, then into the tiles of each row, so every
//                       tile receives its records in ascending (depth, record) order
//   K5                  the tile ranges come from the binning's scan (tile_range); the tile
//                       stage, or k_tile_order, queues the tiles heaviest first
//   K6 k_blend_fwd      per tile: front-to-back compositing, Eq. 11 with clamp/skip/stop
//   K7 k_loss_l1        Eq. 12 (mean L1 colour) + weighted mean L1 depth, its gradient
//   K8 k_blend_bwd2     per (tile, stride) item, back to front: transmittance recovered by
//                       division, per-(pixel, splat) partials of two pixels per lane
//                       (one for tiles of 8) reduced across the wavefront with DPP, summed
//                       per splat in LDS and added with float atomics, splat-major
//   K9 k_project_bwd    per Gaussian, loop over views: chain rule to means, scales,
//                       rotations, opacities and SH coefficients
//
// The per-Gaussian kernels are HBM bound, the blend kernels VALU/transcendental bound; no
// dense contraction, but the entry-by-pixel products of the blend kernels (offsets, colour
// sums) run as rank-1 updates on the matrix cores.
#include "gsr_internal.h"

namespace gsr {
namespace {

// ------------------------------------------------------------------------------------
// wavefront / block helpers (wave64)
// ------------------------------------------------------------------------------------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK,
                                                               0xF, false));
}

// gfx950 lane-half / row swaps: (a, b) -> a's upper 32 lanes exchanged with b's lower 32
// (permlane32), or a's odd 16-lane rows exchanged with b's even rows (permlane16).
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
  a = __builtin_bit_cast(float, int(r[0]));
  b = __builtin_bit_cast(float, int(r[1]));
}
__device__ __forceinline__ void swap_rows(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
  a = __builtin_bit_cast(float, int(r[0]));
  b = __builtin_bit_cast(float, int(r[1]));
}

// Rank-1 update on the matrix cores (v_mfma_f32_4x4x1, one block's A broadcast to all):
// lane l's register i becomes c[i] + A[4 u + i] * b, A[m] being `a` in lane m: four wave-wide
// fused multiply-adds (each rounded once, the bits of fmaf) in one issue slot, with no
// broadcast of A through LDS.  u is a constant in unrolled code.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mfma_rank1(float a, float b, f32x4 c, int u) {
  switch (u) {
    case 0: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 0, 0);
    case 1: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 1, 0);
    case 2: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 2, 0);
    case 3: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 3, 0);
    case 4: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 4, 0);
    case 5: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 5, 0);
    case 6: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 6, 0);
    case 7: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 7, 0);
    case 8: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 8, 0);
    case 9: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 9, 0);
    case 10: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 10, 0);
    case 11: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 11, 0);
    case 12: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 12, 0);
    case 13: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 13, 0);
    case 14: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 14, 0);
    default: return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, 15, 0);
  }
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  for (int off = 32; off > 0; off >>= 1) v = max(v, uint32_t(__shfl_xor(v, off)));
  return v;
}

// Inclusive sum over the wavefront (DPP row shifts, then the rows' totals broadcast to the
// rows behind).  Needs every lane active.
__device__ __forceinline__ uint32_t wave_add_scan(uint32_t v) {
#define GSR_ADD_STEP(CTRL, ROWS) \
  v += uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, ROWS, 0xF, false))
  GSR_ADD_STEP(0x111, 0xF);  // row_shr:1
  GSR_ADD_STEP(0x112, 0xF);
  GSR_ADD_STEP(0x114, 0xF);
  GSR_ADD_STEP(0x118, 0xF);
  GSR_ADD_STEP(0x142, 0xA);  // row_bcast:15
  GSR_ADD_STEP(0x143, 0xC);  // row_bcast:31
#undef GSR_ADD_STEP
  return v;
}

// Between LDS accesses of a wavefront's lanes that read what other lanes wrote: the hardware
// carries out a wavefront's LDS accesses in order, and the fences keep the compiler's (no instruction).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t* red) {
  v = wave_add_scan(v);
  const int nw = blockDim.x >> 6;
  if ((threadIdx.x & 63) == 63) red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t tot = 0;
  for (int i = 0; i < nw; ++i) tot += red[i];
  __syncthreads();
  return tot;
}

__device__ __forceinline__ uint32_t block_exclusive_scan_u32(uint32_t v, uint32_t* red) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t incl = wave_add_scan(v);
  if (lane == 63) red[w] = incl;
  __syncthreads();
  uint32_t pre = 0;
  for (int i = 0; i < w; ++i) pre += red[i];
  return pre + incl - v;
}

// ------------------------------------------------------------------------------------
// Discrete stage.  A fixed sequence of correctly rounded binary32 operations (no fused
// multiply-add: the pragma turns contraction off, divide and square root are built
// correctly rounded) so that culling, splat centre, depth bits and tile rectangle are
// reproducible bit for bit.
// ------------------------------------------------------------------------------------
struct Proj {
  float tx, ty, tz;
  float qw, qx, qy, qz, nq;
  float r[9];  // rotation of the normalised quaternion
  float m[9];  // R diag(s)
  float T[6];  // J W
  float U[6];  // T M
  float a, b, c;  // projected covariance + low-pass
  float txj, tyj;  // the offsets J uses: tx, ty, or +-limit * tz where clamped
  bool clx, cly;   // clamped
  float mux, muy;
  int x0, x1, y0, y1;  // inclusive pixel rectangle
  bool vis;
};

__device__ __forceinline__ void discrete_stage(const float p[3], const float s[3], const float q[4],
                                               const ViewDev& cam, float k, float lowpass, float guard,
                                               float jclamp, Proj& o) {
#pragma clang fp contract(off)
  const float* W = cam.R;
  o.vis = false;
  float tx = W[0] * p[0];
  tx = tx + W[1] * p[1];
  tx = tx + W[2] * p[2];
  tx = tx + cam.t[0];
  float ty = W[3] * p[0];
  ty = ty + W[4] * p[1];
  ty = ty + W[5] * p[2];
  ty = ty + cam.t[1];
  float tz = W[6] * p[0];
  tz = tz + W[7] * p[1];
  tz = tz + W[8] * p[2];
  tz = tz + cam.t[2];
  o.tx = tx;
  o.ty = ty;
  o.tz = tz;
  if (!(tz > cam.znear)) return;
  float nq = q[0] * q[0];
  nq = nq + q[1] * q[1];
  nq = nq + q[2] * q[2];
  nq = nq + q[3] * q[3];
  nq = __builtin_sqrtf(nq);
  o.nq = nq;
  if (!(nq > 0.f)) return;
  const float w = q[0] / nq, x = q[1] / nq, y = q[2] / nq, z = q[3] / nq;
  o.qw = w;
  o.qx = x;
  o.qy = y;
  o.qz = z;
  float* r = o.r;
  r[0] = 1.f - 2.f * (y * y + z * z);
  r[1] = 2.f * (x * y - w * z);
  r[2] = 2.f * (x * z + w * y);
  r[3] = 2.f * (x * y + w * z);
  r[4] = 1.f - 2.f * (x * x + z * z);
  r[5] = 2.f * (y * z - w * x);
  r[6] = 2.f * (x * z - w * y);
  r[7] = 2.f * (y * z + w * x);
  r[8] = 1.f - 2.f * (x * x + y * y);
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j) o.m[i * 3 + j] = r[i * 3 + j] * s[j];
  const float tz2 = tz * tz;
  const float j00 = cam.fx / tz;
  const float j11 = cam.fy / tz;
  // guard-band clamp: an offset beyond jclamp half fields of view enters J as limit * tz
  float txj = tx, tyj = ty;
  o.clx = o.cly = false;
  if (jclamp > 0.f) {
    const float limx = jclamp * ((0.5f * float(cam.W)) / cam.fx);
    const float limy = jclamp * ((0.5f * float(cam.H)) / cam.fy);
    const float ux = tx / tz, uy = ty / tz;
    if (ux < -limx) {
      txj = -limx * tz;
      o.clx = true;
    } else if (ux > limx) {
      txj = limx * tz;
      o.clx = true;
    }
    if (uy < -limy) {
      tyj = -limy * tz;
      o.cly = true;
    } else if (uy > limy) {
      tyj = limy * tz;
      o.cly = true;
    }
  }
  o.txj = txj;
  o.tyj = tyj;
  const float j02 = -(cam.fx * txj) / tz2;
  const float j12 = -(cam.fy * tyj) / tz2;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    o.T[c] = j00 * W[c] + j02 * W[6 + c];
    o.T[3 + c] = j11 * W[3 + c] + j12 * W[6 + c];
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float acc = o.T[i * 3 + 0] * o.m[0 * 3 + c];
      acc = acc + o.T[i * 3 + 1] * o.m[1 * 3 + c];
      acc = acc + o.T[i * 3 + 2] * o.m[2 * 3 + c];
      o.U[i * 3 + c] = acc;
    }
  const float* U = o.U;
  float a = U[0] * U[0];
  a = a + U[1] * U[1];
  a = a + U[2] * U[2];
  a = a + lowpass;
  float b = U[0] * U[3];
  b = b + U[1] * U[4];
  b = b + U[2] * U[5];
  float c = U[3] * U[3];
  c = c + U[4] * U[4];
  c = c + U[5] * U[5];
  c = c + lowpass;
  o.a = a;
  o.b = b;
  o.c = c;
  const float det = a * c - b * b;
  if (!(det > 0.f)) return;
  const float mux = cam.fx * (tx / tz) + cam.cx;
  const float muy = cam.fy * (ty / tz) + cam.cy;
  o.mux = mux;
  o.muy = muy;
  // view frustum: the centre must project inside the image widened by the guard band
  const float gx = guard * float(cam.W), gy = guard * float(cam.H);
  if (!(mux >= -gx && mux <= float(cam.W) + gx && muy >= -gy && muy <= float(cam.H) + gy)) return;
  const float rx = k * __builtin_sqrtf(a);
  const float ry = k * __builtin_sqrtf(c);
  float fx0 = __builtin_ceilf(mux - rx), fx1 = __builtin_floorf(mux + rx);
  float fy0 = __builtin_ceilf(muy - ry), fy1 = __builtin_floorf(muy + ry);
  const float wmax = float(cam.W - 1), hmax = float(cam.H - 1);
  fx0 = (fx0 < 0.f) ? 0.f : fx0;
  fy0 = (fy0 < 0.f) ? 0.f : fy0;
  fx1 = (fx1 > wmax) ? wmax : fx1;
  fy1 = (fy1 > hmax) ? hmax : fy1;
  if (!(fx0 <= fx1 && fy0 <= fy1)) return;
  o.x0 = int(fx0);
  o.x1 = int(fx1);
  o.y0 = int(fy0);
  o.y1 = int(fy1);
  o.vis = true;
}

// Conic (inverse projected covariance); shared by the forward and backward kernels so
// both see identical bits.
__device__ __forceinline__ void conic_of(float a, float b, float c, float& A, float& B, float& C) {
#pragma clang fp contract(off)
  const float det = a * c - b * b;
  const float inv = 1.f / det;
  A = c * inv;
  B = -b * inv;
  C = a * inv;
}

// Exact tile culling: the tile columns [lo, hi] of tile row ty (local) that the ellipse
// d^T Q d <= k^2 of a splat can reach within the row's pixel band, Q = (A, B; B, C) its
// binary32 conic.  Over the band's offsets [u0, u1] from the centre, the boundary's
// rightmost point lies at dy = clamp(-B k / sqrt(C det_Q), u0, u1) and the leftmost at
// dy = clamp(B k / sqrt(C det_Q), u0, u1), with x offsets (+-sqrt(max(0, A k^2 - det_Q
// dy^2)) - B dy) / A; the pixels between ceil and floor of the two edges, kept inside the
// rectangle's columns, name the tiles.  One correctly rounded operation per line (the
// kernels compile with contraction off here), so the lists are reproducible bit for bit;
// a degenerate conic or a NaN keeps the rectangle's columns.  False when the row keeps
// no tile.
// The row-independent part of row_run: det_Q, the boundary's extreme offset B k / sqrt(C
// det_Q) and A k^2; `whole` when the conic is degenerate (or a NaN): keep the rectangle.
struct RowCut {
  float dq, q, ak;
  bool whole;
};

__device__ __forceinline__ RowCut row_cut(float A, float B, float C, float k) {
#pragma clang fp contract(off)
  RowCut r{};
  r.dq = A * C - B * B;
  r.whole = true;
  if (!(r.dq > 0.f)) return r;
  const float sq = __builtin_sqrtf(C * r.dq);
  if (!(sq > 0.f)) return r;
  r.q = (B * k) / sq;
  r.ak = A * (k * k);
  r.whole = false;
  return r;
}

// row_run for tile row ty given the record's row_cut; ts = 1 << tshift
__device__ __forceinline__ bool row_run_at(const RowCut& rc, float mux, float muy, float A, float B, int ts,
                                           int tshift, int ty, int W, int H, int tx0, int tx1, int& lo, int& hi) {
#pragma clang fp contract(off)
  lo = tx0;
  hi = tx1;
  if (rc.whole) return true;
  const float dyr = -rc.q, dyl = rc.q;
  const int ylast = min(ty * ts + ts - 1, H - 1);
  const float u0 = float(ty * ts) - muy;
  const float u1 = float(ylast) - muy;
  const float ur = fminf(fmaxf(dyr, u0), u1);
  const float ul = fminf(fmaxf(dyl, u0), u1);
  const float sr = __builtin_sqrtf(fmaxf(rc.ak - rc.dq * (ur * ur), 0.f));
  const float xr = (sr - B * ur) / A;
  const float sl = __builtin_sqrtf(fmaxf(rc.ak - rc.dq * (ul * ul), 0.f));
  const float xl = ((-sl) - B * ul) / A;
  float pl = ceilf(mux + xl);
  float pr = floorf(mux + xr);
  const float xa = float(tx0 * ts);
  const float xb = float(min(tx1 * ts + ts - 1, W - 1));
  if (!(pl >= xa)) pl = xa;  // also a NaN
  if (!(pr <= xb)) pr = xb;
  if (!(pl <= pr)) return false;
  lo = int(pl) >> tshift;  // pl, pr >= 0 here
  hi = int(pr) >> tshift;
  return true;
}

__device__ __forceinline__ bool row_run(float mux, float muy, float A, float B, float C, float k, int ts, int ty,
                                        int W, int H, int tx0, int tx1, int& lo, int& hi) {
  return row_run_at(row_cut(A, B, C, k), mux, muy, A, B, ts, __builtin_ctz(unsigned(ts)), ty, W, H, tx0, tx1, lo,
                    hi);
}

// Splat value a = o * exp(-q/2), q = A dx^2 + 2 B dx dy + C dy^2.  The compositing kernels
// stage each record with its conic scaled by -log2(e)/2, (a', b', c') = (A, 2B, C) * k,
// so that exp(-q/2) = exp2(q') with q' = (a' dx + b' dy) dx + c' dy^2: five operations and
// one exp2.  One fixed instruction sequence, so the forward skip decision and its
// recomputation in the backward agree bitwise.
constexpr float kNegHalfLog2e = -0.72134752044448170368f;  // -log2(e) / 2

__device__ __forceinline__ float splat_alpha(float dx, float dy, float ap, float bp, float cp, float o, float& G) {
#pragma clang fp contract(off)
  const float q = __builtin_fmaf(__builtin_fmaf(ap, dx, bp * dy), dx, (cp * dy) * dy);
  G = __builtin_amdgcn_exp2f(q);
  return o * G;
}

// Record id as the compositing kernels stage it: the centre, (a', b', c', opacity) as above and
// (colour, depth).
__device__ __forceinline__ void stage_record(const Records& rec, uint32_t id, float& mx, float& my, float4& sq,
                                             float4& col) {
  const float4 g0 = rec.r0[id], g1 = rec.r1[id], c = rec.rgb[id];
  mx = g0.x;
  my = g0.y;
  sq = make_float4(kNegHalfLog2e * g0.z, (2.f * kNegHalfLog2e) * g0.w, kNegHalfLog2e * g1.x, g1.y);
  col = make_float4(c.x, c.y, c.z, g1.z);
}

// ------------------------------------------------------------------------------------
// Real spherical harmonics, orthonormal with Condon-Shortley phase, as Cartesian
// polynomials of the unit direction (x, y, z).  Constants are N_l^m (and sqrt 2 for
// m != 0) times the Legendre factors:
//   l=0: 1/(2 sqrt(pi))
//   l=1: sqrt(3/(4 pi))                          -> -y, z, -x
//   l=2: sqrt(15/(4 pi)) xy, -..yz, sqrt(5/(16 pi))(3z^2-1), -..xz, sqrt(15/(16 pi))(x^2-y^2)
//   l=3: sqrt(35/(32 pi)), sqrt(105/(4 pi)), sqrt(21/(32 pi)), sqrt(7/(16 pi)), sqrt(105/(16 pi))
// Gradients are those of these polynomials; the chain rule through the normalisation
// of the direction removes their radial part.
// ------------------------------------------------------------------------------------
constexpr float kY00 = 0.28209479177387814f;   // 1/(2 sqrt(pi))
constexpr float kY1 = 0.4886025119029199f;     // sqrt(3/(4 pi))
constexpr float kY2a = 1.0925484305920792f;    // sqrt(15/(4 pi))
constexpr float kY2b = 0.31539156525252005f;   // sqrt(5/(16 pi))
constexpr float kY2c = 0.5462742152960396f;    // sqrt(15/(16 pi))
constexpr float kY3a = 0.5900435899266435f;    // sqrt(35/(32 pi))
constexpr float kY3b = 2.890611442640554f;     // sqrt(105/(4 pi))
constexpr float kY3c = 0.4570457994644658f;    // sqrt(21/(32 pi))
constexpr float kY3d = 0.3731763325901154f;    // sqrt(7/(16 pi))
constexpr float kY3e = 1.445305721320277f;     // sqrt(105/(16 pi))

template <int DEG>
__device__ __forceinline__ void sh_basis(float x, float y, float z, float* Y) {
  Y[0] = kY00;
  if (DEG >= 1) {
    Y[1] = -kY1 * y;
    Y[2] = kY1 * z;
    Y[3] = -kY1 * x;
  }
  if (DEG >= 2) {
    Y[4] = kY2a * x * y;
    Y[5] = -kY2a * y * z;
    Y[6] = kY2b * (3.f * z * z - 1.f);
    Y[7] = -kY2a * x * z;
    Y[8] = kY2c * (x * x - y * y);
  }
  if (DEG >= 3) {
    Y[9] = -kY3a * y * (3.f * x * x - y * y);
    Y[10] = kY3b * x * y * z;
    Y[11] = -kY3c * y * (5.f * z * z - 1.f);
    Y[12] = kY3d * z * (5.f * z * z - 3.f);
    Y[13] = -kY3c * x * (5.f * z * z - 1.f);
    Y[14] = kY3e * z * (x * x - y * y);
    Y[15] = -kY3a * x * (x * x - 3.f * y * y);
  }
}

// d/d(x,y,z) of the basis polynomials, contracted with weights w[k]: out = sum_k w_k grad Y_k.
template <int DEG>
__device__ __forceinline__ void sh_grad_dot(float x, float y, float z, const float* w, float out[3]) {
  float gx = 0.f, gy = 0.f, gz = 0.f;
  if (DEG >= 1) {
    gy += -kY1 * w[1];
    gz += kY1 * w[2];
    gx += -kY1 * w[3];
  }
  if (DEG >= 2) {
    gx += kY2a * y * w[4];
    gy += kY2a * x * w[4];
    gy += -kY2a * z * w[5];
    gz += -kY2a * y * w[5];
    gz += 6.f * kY2b * z * w[6];
    gx += -kY2a * z * w[7];
    gz += -kY2a * x * w[7];
    gx += 2.f * kY2c * x * w[8];
    gy += -2.f * kY2c * y * w[8];
  }
  if (DEG >= 3) {
    gx += -6.f * kY3a * x * y * w[9];
    gy += -kY3a * (3.f * x * x - 3.f * y * y) * w[9];
    gx += kY3b * y * z * w[10];
    gy += kY3b * x * z * w[10];
    gz += kY3b * x * y * w[10];
    gy += -kY3c * (5.f * z * z - 1.f) * w[11];
    gz += -10.f * kY3c * y * z * w[11];
    gz += kY3d * (15.f * z * z - 3.f) * w[12];
    gx += -kY3c * (5.f * z * z - 1.f) * w[13];
    gz += -10.f * kY3c * x * z * w[13];
    gx += 2.f * kY3e * x * z * w[14];
    gy += -2.f * kY3e * y * z * w[14];
    gz += kY3e * (x * x - y * y) * w[14];
    gx += -kY3a * (3.f * x * x - 3.f * y * y) * w[15];
    gy += 6.f * kY3a * x * y * w[15];
  }
  out[0] = gx;
  out[1] = gy;
  out[2] = gz;
}

// ------------------------------------------------------------------------------------
// K1: projection.  Per view, the block also sums its tile counts and visible records.
// ------------------------------------------------------------------------------------
template <int DEG>
__global__ __launch_bounds__(kProjThreads) void k_project(GaussDev g, ViewTable vt, Rules ru, int tile,
                                                          Records rec, uint2* blocksums, int nblk,
                                                          float* zero_rows, uint32_t* ctrl, int clear_words,
                                                          float exact_k) {
  constexpr int K = (DEG + 1) * (DEG + 1);
  __shared__ uint32_t red[kProjThreads / 64];
  // the step's control words start at zero (no kernel before the projection reads them)
  if (blockIdx.x == 0 && int(threadIdx.x) < clear_words) ctrl[threadIdx.x] = 0u;
  const int64_t gi = int64_t(blockIdx.x) * kProjThreads + threadIdx.x;
  const bool valid = gi < g.n;
  float p[3] = {0.f, 0.f, 0.f}, s[3] = {1.f, 1.f, 1.f}, q[4] = {1.f, 0.f, 0.f, 0.f}, op = 0.f;
  float sh[K * 3];
  if (valid) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      p[i] = g.means[gi * 3 + i];
      s[i] = g.scales[gi * 3 + i];
    }
    const float4 q4 = reinterpret_cast<const float4*>(g.quats)[gi];
    q[0] = q4.x;
    q[1] = q4.y;
    q[2] = q4.z;
    q[3] = q4.w;
    op = g.opac[gi];
  }
  // the colour coefficients are read at the first view that sees the Gaussian (none for
  // a Gaussian outside every view)
  bool have_sh = false;
#pragma unroll
  for (int i = 0; i < K * 3; ++i) sh[i] = 0.f;
  for (int v = 0; v < vt.nviews; ++v) {
    const ViewDev& cam = vt.v[v];
    uint32_t cnt = 0;
    if (valid) {
      Proj pr;
      discrete_stage(p, s, q, cam, ru.k, ru.lowpass, ru.guard, ru.jclamp, pr);
      const int64_t rid = int64_t(v) * g.n + gi;
      if (pr.vis) {
        if (!have_sh) {
          const float* src = g.sh + gi * (K * 3);
#pragma unroll
          for (int i = 0; i < K * 3; ++i) sh[i] = src[i];
          have_sh = true;
        }
        const int tx0 = pr.x0 / tile, tx1 = pr.x1 / tile, ty0 = pr.y0 / tile, ty1 = pr.y1 / tile;
        cnt = uint32_t((tx1 - tx0 + 1) * (ty1 - ty0 + 1));
        float A, B, C;
        conic_of(pr.a, pr.b, pr.c, A, B, C);
        float d0 = p[0] - cam.cam_pos[0], d1 = p[1] - cam.cam_pos[1], d2 = p[2] - cam.cam_pos[2];
        const float inv = 1.f / __builtin_sqrtf(d0 * d0 + d1 * d1 + d2 * d2);
        float Y[K];
        sh_basis<DEG>(d0 * inv, d1 * inv, d2 * inv, Y);
        float col[3];
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
          float acc = 0.5f;
#pragma unroll
          for (int kk = 0; kk < K; ++kk) acc += sh[kk * 3 + ch] * Y[kk];
          col[ch] = acc > 0.f ? acc : 0.f;
        }
        rec.r0[rid] = make_float4(pr.mux, pr.muy, A, B);
        rec.r1[rid] = make_float4(C, op, pr.tz, 0.f);
        rec.rgb[rid] = make_float4(col[0], col[1], col[2], 0.f);
        rec.rect[rid] = make_uint2(uint32_t(tx0) | (uint32_t(tx1) << 16), uint32_t(ty0) | (uint32_t(ty1) << 16));
        if (rec.runs) {  // exact tiles: the column runs of the first kRowRuns tile rows, once per record
          const RowCut rc = row_cut(A, B, C, exact_k);
          const int tshift = __builtin_ctz(unsigned(tile));
          uint32_t rr[kRowRuns];
#pragma unroll
          for (int k = 0; k < kRowRuns; ++k) {
            rr[k] = kRunEmpty;
            if (k <= ty1 - ty0) {
              int lo, hi;
              if (row_run_at(rc, pr.mux, pr.muy, A, B, tile, tshift, ty0 + k, cam.W, cam.H, tx0, tx1, lo, hi))
                rr[k] = uint32_t(lo) | (uint32_t(hi) << 16);
            }
          }
          uint4* dst = reinterpret_cast<uint4*>(rec.runs + rid * kRowRuns);
#pragma unroll
          for (int k = 0; k < kRowRuns / 4; ++k) dst[k] = make_uint4(rr[4 * k], rr[4 * k + 1], rr[4 * k + 2], rr[4 * k + 3]);
        }
        if (zero_rows) {  // the backward's 2D-gradient row of this record starts at zero
          float4* z = reinterpret_cast<float4*>(zero_rows + rid * kGrad2D);
          z[0] = make_float4(0.f, 0.f, 0.f, 0.f);
          z[1] = make_float4(0.f, 0.f, 0.f, 0.f);
          z[2] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
      }
      rec.counts[rid] = cnt;
    }
    const uint32_t bs = block_sum_u32(cnt, red);
    const uint32_t bv = block_sum_u32(cnt ? 1u : 0u, red);
    if (threadIdx.x == 0) blocksums[int64_t(v) * nblk + blockIdx.x] = make_uint2(bs, bv);
  }
}

// ------------------------------------------------------------------------------------
// K2: exclusive scans of per-block sums (one block of 1024 threads).  Totals are written
// as 64-bit values; consumers clamp them to their buffer capacity.
// ------------------------------------------------------------------------------------
template <int NT>
__device__ __forceinline__ unsigned long long block_inclusive_scan_u64(unsigned long long v, unsigned long long* part) {
  const int t = threadIdx.x;
  part[t] = v;
  __syncthreads();
  for (int off = 1; off < NT; off <<= 1) {
    const unsigned long long add = t >= off ? part[t - off] : 0ull;
    __syncthreads();
    part[t] += add;
    __syncthreads();
  }
  return part[t];
}

// Writes the totals, and to the host's pinned copy where there is one (read after a
// synchronisation of the stream; a copy of the two words took the host and the stream longer than
// the scan).
__device__ __forceinline__ void store_totals(unsigned long long x, unsigned long long y, unsigned long long* totals,
                                             unsigned long long* host) {
  totals[0] = x;
  totals[1] = y;
  if (host) {
    __hip_atomic_store(host, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(host + 1, y, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

__global__ __launch_bounds__(1024) void k_scan_pairs(uint2* a, int count, unsigned long long* totals,
                                                     unsigned long long* host) {
  __shared__ unsigned long long part[1024];
  const int t = threadIdx.x;
  const int per = (count + 1023) / 1024;
  const int beg = min(count, t * per), end = min(count, beg + per);
  unsigned long long sx = 0, sy = 0;
  for (int i = beg; i < end; ++i) {
    const uint2 x = a[i];
    sx += x.x;
    sy += x.y;
  }
  const unsigned long long ix = block_inclusive_scan_u64<1024>(sx, part);
  __syncthreads();
  const unsigned long long iy = block_inclusive_scan_u64<1024>(sy, part);
  unsigned long long rx = ix - sx, ry = iy - sy;
  for (int i = beg; i < end; ++i) {
    const uint2 x = a[i];
    a[i] = make_uint2(uint32_t(rx), uint32_t(ry));
    rx += x.x;
    ry += x.y;
  }
  if (t == 1023) store_totals(ix, iy, totals, host);
}

__global__ __launch_bounds__(1024) void k_scan_u32(uint32_t* a, int count, unsigned long long* total) {
  __shared__ unsigned long long part[1024];
  const int t = threadIdx.x;
  const int per = (count + 1023) / 1024;
  const int beg = min(count, t * per), end = min(count, beg + per);
  unsigned long long sum = 0;
  for (int i = beg; i < end; ++i) sum += a[i];
  const unsigned long long incl = block_inclusive_scan_u64<1024>(sum, part);
  unsigned long long run = incl - sum;
  for (int i = beg; i < end; ++i) {
    const uint32_t x = a[i];
    a[i] = uint32_t(run);
    run += x;
  }
  if (t == 1023) *total = incl;
}

// The same scan of more than kSumMany pairs, in place, by tiles of kSumTile: their sums, then each
// block adds up the sums in front of its tile and scans it.  One block over all 188k block sums
// of sixteen views of 3M Gaussians took 336 us and over the 15k of eight views of 500k 32 us;
// the two launches take 11 and 10.  With fewer the second launch costs what it saves.  part: a
// tile's pairs and records as 64-bit sums (its 65,536 records can cover 2^20 tiles each, and a
// total past 2^32 has to show).
constexpr int kSumTile = 256;
constexpr int64_t kSumMany = 4096;

__global__ __launch_bounds__(kSumTile) void k_sum_pairs(const uint2* a, int64_t count, unsigned long long* part) {
  __shared__ uint32_t red[kSumTile / 64];
  __shared__ unsigned long long red64[kSumTile / 64];
  const int64_t i = int64_t(blockIdx.x) * kSumTile + threadIdx.x;
  const uint2 v = i < count ? a[i] : make_uint2(0u, 0u);
  unsigned long long x = v.x;
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  if ((threadIdx.x & 63) == 0) red64[threadIdx.x >> 6] = x;
  const uint32_t y = block_sum_u32(v.y, red);  // (its barrier also publishes red64)
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = (red64[0] + red64[1]) + (red64[2] + red64[3]);
    part[2 * blockIdx.x + 1] = y;
  }
}

__global__ __launch_bounds__(kSumTile) void k_scan_pairs_down(uint2* a, int64_t count, const unsigned long long* part,
                                                              unsigned long long* totals, unsigned long long* host) {
  __shared__ unsigned long long red[kSumTile];
  const int t = threadIdx.x;
  unsigned long long bx = 0, by = 0;
  for (int i = t; i < int(blockIdx.x); i += kSumTile) {
    bx += part[2 * i];
    by += part[2 * i + 1];
  }
  const int64_t i = int64_t(blockIdx.x) * kSumTile + t;
  const uint2 v = i < count ? a[i] : make_uint2(0u, 0u);
  (void)block_inclusive_scan_u64<kSumTile>(bx, red);
  const unsigned long long x0 = red[kSumTile - 1];
  __syncthreads();
  (void)block_inclusive_scan_u64<kSumTile>(by, red);
  const unsigned long long y0 = red[kSumTile - 1];
  __syncthreads();
  const unsigned long long ix = x0 + block_inclusive_scan_u64<kSumTile>(v.x, red);
  __syncthreads();
  const unsigned long long iy = y0 + block_inclusive_scan_u64<kSumTile>(v.y, red);
  if (i < count) a[i] = make_uint2(uint32_t(ix - v.x), uint32_t(iy - v.y));
  if (i == count - 1) store_totals(ix, iy, totals, host);
}

// Flags a capacity overflow: the step's word and the sticky copy next to it.
__device__ __forceinline__ void raise_overflow(uint32_t* overflow) {
  atomicOr(overflow, 1u);
  atomicOr(overflow + (kOverflowSticky - kOverflow), 1u);
}

// A device-side count clamped to the capacity the grid and buffers were sized for; zero
// once a capacity overflow has been flagged, so that nothing downstream of an overflow
// reads partially written buffers.
__device__ __forceinline__ uint32_t clamp_count(const unsigned long long* count, int64_t cap,
                                                const uint32_t* overflow) {
  if (*overflow) return 0u;
  const unsigned long long c = *count;
  return uint32_t(c < (unsigned long long)cap ? c : (unsigned long long)cap);
}

// ------------------------------------------------------------------------------------
// K3a: compaction of the visible records into (depth bits, record id) pairs, record order
// ------------------------------------------------------------------------------------
// raw: the block sums are the projection's, not scanned (at most kSumMany of them):
// each block adds the visible records of the blocks in front of it itself, and the last
// block writes the totals (pairs, visible records) to totals[0..1].  Otherwise they were
// scanned (launch_scan_pairs, which wrote the totals).  vstart[0 .. views]: where each view's
// records start, and their end.
__global__ __launch_bounds__(kProjThreads) void k_compact(int64_t n, Records rec, const uint2* blocksums, int nblk,
                                                          unsigned long long* totals, int64_t cap_M,
                                                          uint32_t* dkeys, uint32_t* dvals, int64_t cap,
                                                          uint32_t* overflow, int raw, uint32_t* vstart) {
  __shared__ uint32_t red[kProjThreads / 64];
  __shared__ unsigned long long red64[kProjThreads / 64];
  const int v = blockIdx.y;
  const int64_t me = int64_t(v) * nblk + blockIdx.x;  // this block's sums
  const int64_t nb = int64_t(gridDim.y) * nblk;
  const int64_t gi = int64_t(blockIdx.x) * kProjThreads + threadIdx.x;
  const int64_t rid = int64_t(v) * n + gi;
  const uint32_t vis = (gi < n && rec.counts[rid] != 0u) ? 1u : 0u;
  uint32_t base;
  if (raw) {
    uint32_t before = 0;
    for (int64_t i = threadIdx.x; i < me; i += kProjThreads) before += blocksums[i].y;
    base = block_sum_u32(before, red);
    if (me == nb - 1) {  // block-uniform: the last block writes the totals
      unsigned long long px = 0;
      for (int64_t i = threadIdx.x; i < nb; i += kProjThreads) px += blocksums[i].x;
      for (int off = 32; off > 0; off >>= 1) px += __shfl_xor(px, off);
      if ((threadIdx.x & 63) == 0) red64[threadIdx.x >> 6] = px;
      const uint32_t mine = block_sum_u32(vis, red);  // (its barrier also publishes red64)
      if (threadIdx.x == 0) {
        unsigned long long pairs = 0;
        for (int i = 0; i < kProjThreads / 64; ++i) pairs += red64[i];
        totals[0] = pairs;
        totals[1] = (unsigned long long)base + mine;
        if (pairs > (unsigned long long)cap_M) raise_overflow(overflow);
      }
    }
  } else {
    base = blocksums[me].y;
    // more (tile, record) pairs than the binning buffers hold: flag it before anything
    // reads the flag (every later kernel then sees zero records)
    if (me == 0 && threadIdx.x == 0 && totals[0] > (unsigned long long)cap_M) raise_overflow(overflow);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) vstart[v] = base;  // the view's first place
  const uint32_t excl = block_exclusive_scan_u32(vis, red);
  if (me == nb - 1 && threadIdx.x == kProjThreads - 1) vstart[gridDim.y] = base + excl + vis;
  if (!vis) return;
  const uint32_t off = base + excl;
  if (int64_t(off) >= cap) {
    raise_overflow(overflow);
    return;
  }
  dkeys[off] = __float_as_uint(rec.r1[rid].z);
  dvals[off] = uint32_t(rid);
}

// ------------------------------------------------------------------------------------
// K4: stable LSD radix sort of (u32 key, u32 value) by 8-bit digits, each view's
// keys by themselves (the compaction leaves them in view order, and a tile's list needs no
// order between views; records in view order let the binning handle one view's tile rows at
// a time).  A key tile is ITEMS keys a thread of one view; counts are read from the device
// (clamped to the capacity the grid was sized for).  Per pass:
//   hist:    per-tile digit histograms
//   rowscan: (views of more than kSortFold tiles, histograms digit-major [256][ntile]) one block
//            per digit scans its row -> keys of the digit in front of each tile, and the digit total.
//            With fewer the histograms are tile-major [ntile][256] and each block of the
//            scatter adds up its view's itself: a launch less
//   scatter: each block ranks its keys stably, orders them in LDS, and writes them out in
//            runs: a key's slot is the view's start, its keys of smaller digits, the digit's keys
//            in the view's tiles in front and its rank in the tile
// A wavefront owns 64 ITEMS consecutive keys, so that it ranks them by itself (peers of a
// digit by ballots, a counter per digit of its own in LDS), and the block meets at a barrier
// only to add up the wavefronts' counters (four rounds of 256 keys with two barriers each, and
// a store per key, before).  Views of up to kSmallMost keys are sorted by one block each, in LDS,
// all passes in one launch.
// Kernel trace of a whole sort, before -> after: 1.9k keys 43 -> 13 us, 12k 49 -> 41, 85k 51 -> 39,
// 335k 73 -> 51 (captured), 1M 103 -> 70, 2.7M in eight views 231 -> 126.  The small ones are
// chains of latencies (2 us of each launch), the large ones VALU issue of the ranking (half) and
// the scattered writes.
// ------------------------------------------------------------------------------------
// 8-bit digits: wider ones (11 bits, three passes for a depth key) ran slower on MI355X,
// their histograms being written and read across many more cache lines
constexpr int kSortBits = 8, kSortDigits = 1 << kSortBits;
constexpr int kSortThreads = 1024, kSortWaves = kSortThreads / 64;
// Keys of a thread: 4 (tiles of 4,096), or 2 where that still folds: 85k keys sort in 39 us with
// 2 and 49 with 4, 335k in 51 and 55, eight views of 340k in 170 and 126.
constexpr int kSortItems = 4, kSortItemsFew = 2;
// A view's tiles up to which the scatter adds up the histograms itself: at 102 tiles a captured sort
// takes 55 us with it and 70 with the row scans, at 162 61 and 63, at 245 75 and 70.
constexpr int kSortFold = 224;
constexpr int64_t kSmallMost = 16 * kSortThreads;

// Block b of a grid of G blocks (G a multiple of 8) as index (b mod 8) * (G / 8) + b / 8:
// the hardware hands consecutive blocks to the eight XCDs in turn, so with this index
// consecutive key tiles and record chunks run on one XCD, and the strided count words
// they share meet in that XCD's L2.  (Only for even work: the row-list segments stay
// round-robin, as a contiguous range of rows would load some XCDs far more than others.)
__device__ __forceinline__ int xcd_block(int b, int G) { return (b & 7) * (G >> 3) + (b >> 3); }
static int xcd_grid(int64_t blocks) { return int((blocks + 7) / 8 * 8); }

// The keys of tile tb: its view's first key and end (in the key arrays), this tile's first key, the view's
// first tile and the next view's (ntile: past the last).  False past the last tile.
struct SortTile {
  uint32_t vbeg, vend, beg;
  int t0, t1;
};
// (every lane active; lane v looks up view v, all loads in flight together)
template <int ITEMS>
__device__ __forceinline__ bool sort_tile(const uint32_t* vstart, int views, const unsigned long long* count, int64_t cap,
                                          const uint32_t* overflow, int tb, SortTile& o) {
  static_assert(GSR_MAX_VIEWS <= 16, "a view per lane of a DPP row");
  constexpr uint32_t kTile = ITEMS * kSortThreads;
  const int lane = threadIdx.x & 63;
  const uint32_t a = vstart[min(lane, views)], b = vstart[min(lane + 1, views)];
  const unsigned long long c = *count;
  const uint32_t over = *overflow;
  const uint32_t M = over ? 0u : uint32_t(c < (unsigned long long)cap ? c : (unsigned long long)cap);
  const uint32_t beg = min(a, M), end = min(b, M);  // (empty past the last view)
  const uint32_t tiles = (end - beg + kTile - 1) / kTile;
  uint32_t incl = tiles;
#define GSR_ADD_STEP(CTRL) incl += uint32_t(__builtin_amdgcn_update_dpp(0, int(incl), CTRL, 0xF, 0xF, false))
  GSR_ADD_STEP(0x111);  // row_shr:1
  GSR_ADD_STEP(0x112);
  GSR_ADD_STEP(0x114);
  GSR_ADD_STEP(0x118);
#undef GSR_ADD_STEP
  const uint64_t past = __ballot(lane < views && uint32_t(tb) < incl);
  if (past == 0) return false;
  const int v = __builtin_ctzll(past);
  o.vbeg = uint32_t(__builtin_amdgcn_readlane(int(beg), v));
  o.vend = uint32_t(__builtin_amdgcn_readlane(int(end), v));
  o.t1 = __builtin_amdgcn_readlane(int(incl), v);
  o.t0 = o.t1 - __builtin_amdgcn_readlane(int(tiles), v);
  o.beg = o.vbeg + uint32_t(tb - o.t0) * kTile;
  return true;
}

template <int ITEMS, bool FOLD>
__global__ __launch_bounds__(kSortThreads) void k_radix_hist(const uint32_t* keys, const uint32_t* vstart, int views,
                                                             const unsigned long long* count, int64_t cap,
                                                             const uint32_t* overflow, int shift, uint32_t* hist,
                                                             int nblk) {
  __shared__ uint32_t h[kSortDigits];
  const int t = threadIdx.x;
  const int tb = xcd_block(blockIdx.x, gridDim.x);  // this block's tile of keys
  if (tb >= nblk) return;                            // block-uniform
  if (t < kSortDigits) h[t] = 0;
  __syncthreads();
  SortTile st;
  if (sort_tile<ITEMS>(vstart, views, count, cap, overflow, tb, st)) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint32_t idx = st.beg + uint32_t(i * kSortThreads + t);
      if (idx < st.vend) atomicAdd(&h[(keys[idx] >> shift) & (kSortDigits - 1)], 1u);
    }
  }
  __syncthreads();
  if (t < kSortDigits) hist[FOLD ? int64_t(tb) * kSortDigits + t : int64_t(t) * nblk + tb] = h[t];
}

__global__ __launch_bounds__(256) void k_radix_rowscan(uint32_t* hist, int nblk, uint32_t* digit_tot) {
  __shared__ uint32_t red[4];
  __shared__ uint32_t carry;
  uint32_t* row = hist + int64_t(blockIdx.x) * nblk;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int start = 0; start < nblk; start += 256) {
    const int i = start + threadIdx.x;
    const uint32_t v = i < nblk ? row[i] : 0u;
    const uint32_t ex = block_exclusive_scan_u32(v, red);
    const uint32_t c = carry;
    if (i < nblk) row[i] = c + ex;
    __syncthreads();
    if (threadIdx.x == 255) carry = c + ex + v;
    __syncthreads();
  }
  if (threadIdx.x == 0) digit_tot[blockIdx.x] = carry;
}

// Ranks a wavefront's 64 ITEMS keys within their digits, in order (row r of 64 keys at a time):
// rank[r], and in cnt (the wavefront's own counters) its keys of each digit.
template <int ITEMS>
__device__ __forceinline__ void wave_rank(const uint32_t (&key)[ITEMS], int shift, uint16_t* cnt,
                                          uint16_t (&rank)[ITEMS]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < kSortDigits / 64; ++i) cnt[64 * i + lane] = 0;
  wave_lds_sync();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t d = (key[r] >> shift) & (kSortDigits - 1);
    uint32_t lo = ~0u, hi = ~0u;  // the lanes with this lane's digit
#pragma unroll
    for (int bit = 0; bit < kSortBits; ++bit) {
      const uint64_t m = __ballot((d >> bit) & 1u);
      const uint32_t other = ((d >> bit) & 1u) - 1u;  // all bits where the lane's own bit is clear
      lo &= uint32_t(m) ^ other;
      hi &= uint32_t(m >> 32) ^ other;
    }
    const uint32_t in = __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
    const uint32_t prior = cnt[d];
    rank[r] = uint16_t(prior + in);
    wave_lds_sync();
    if (in == 0) cnt[d] = uint16_t(prior + __popc(lo) + __popc(hi));
    wave_lds_sync();
  }
}

// By the first 256 threads, digit t each: the wavefronts' counters become offsets within the digit;
// returns the tile's keys of digit t.
__device__ __forceinline__ uint32_t digit_offsets(uint16_t (*cnt)[kSortDigits], int t) {
  uint32_t c[kSortWaves], run = 0;
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) c[w] = cnt[w][t];
#pragma unroll
  for (int w = 0; w < kSortWaves; ++w) {
    cnt[w][t] = uint16_t(run);
    run += c[w];
  }
  return run;
}

// Exclusive scans over the 256 digits of two values of the first 256 threads (called by all;
// red: 8 words; one barrier inside).
__device__ __forceinline__ void digit_scan2(uint32_t a, uint32_t b, uint32_t* red, uint32_t& ea, uint32_t& eb) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t ia = a, ib = b;
  if (w < kSortDigits / 64) {  // wave-uniform
    ia = wave_add_scan(a);
    ib = wave_add_scan(b);
    if (lane == 63) {
      red[w] = ia;
      red[4 + w] = ib;
    }
  }
  __syncthreads();
  if (w < kSortDigits / 64)
    for (int i = 0; i < w; ++i) {
      ia += red[i];
      ib += red[4 + i];
    }
  ea = ia - a;
  eb = ib - b;
}

template <int ITEMS, bool FOLD>
__global__ __launch_bounds__(kSortThreads) void k_radix_scatter(const uint32_t* kin, const uint32_t* vin,
                                                                uint32_t* kout, uint32_t* vout,
                                                                const uint32_t* vstart, int views,
                                                                const unsigned long long* count, int64_t cap,
                                                                const uint32_t* overflow, int shift,
                                                                const uint32_t* hist, const uint32_t* digit_tot,
                                                                int nblk) {
  __shared__ uint16_t cnt[kSortWaves][kSortDigits];
  constexpr int kTile = ITEMS * kSortThreads;
  __shared__ uint32_t s_key[kTile], s_val[kTile];
  __shared__ uint32_t lbase[kSortDigits], delta[kSortDigits], red[8];
  constexpr int G = kSortThreads / kSortDigits;  // FOLD: threads that add up one digit's histograms
  static_assert(kTile >= G * kSortDigits, "s_key and s_val hold the partial sums first");
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int tb = xcd_block(blockIdx.x, gridDim.x);  // this block's tile of keys
  if (tb >= nblk) return;                            // block-uniform
  SortTile st;
  if (!sort_tile<ITEMS>(vstart, views, count, cap, overflow, tb, st)) return;  // block-uniform
  // the keys past the view's end are all bits: last in the tile, and not written
  uint32_t key[ITEMS], val[ITEMS];
  const uint32_t first = st.beg + uint32_t(w * 64 * ITEMS + lane);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t idx = first + uint32_t(64 * r);
    key[r] = idx < st.vend ? kin[idx] : ~0u;
    val[r] = idx < st.vend ? vin[idx] : 0u;
  }
  // the view's keys of each digit, and those of its tiles in front
  uint32_t tot = 0, pre = 0;
  if (FOLD) {
    const uint32_t* h = hist + (t & (kSortDigits - 1));
#pragma unroll 8
    for (int i = st.t0 + t / kSortDigits; i < st.t1; i += G) {
      const uint32_t c = h[int64_t(i) * kSortDigits];
      tot += c;
      pre += i < tb ? c : 0u;
    }
    s_key[t] = tot;
    s_val[t] = pre;
  } else if (t < kSortDigits) {
    const uint32_t* row = hist + int64_t(t) * nblk;
    const uint32_t before = row[st.t0];
    tot = (st.t1 < nblk ? row[st.t1] : digit_tot[t]) - before;
    pre = row[tb] - before;
  }
  uint16_t rank[ITEMS];
  wave_rank(key, shift, cnt[w], rank);
  __syncthreads();
  uint32_t own = 0;
  if (t < kSortDigits) {
    if (FOLD)
#pragma unroll
      for (int i = 1; i < G; ++i) {
        tot += s_key[i * kSortDigits + t];
        pre += s_val[i * kSortDigits + t];
      }
    own = digit_offsets(cnt, t);
  }
  uint32_t slot, at;
  digit_scan2(tot, own, red, slot, at);
  if (t < kSortDigits) {
    lbase[t] = at;
    delta[t] = st.vbeg + slot + pre - at;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t d = (key[r] >> shift) & (kSortDigits - 1);
    const uint32_t i = lbase[d] + cnt[w][d] + rank[r];
    s_key[i] = key[r];
    s_val[i] = val[r];
  }
  __syncthreads();
  const uint32_t n = min(st.vend - st.beg, uint32_t(kTile));
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t i = uint32_t(r * kSortThreads + t);
    if (i < n) {
      const uint32_t k = s_key[i];
      const uint32_t dst = delta[(k >> shift) & (kSortDigits - 1)] + i;
      kout[dst] = k;
      vout[dst] = s_val[i];
    }
  }
}

// The whole sort of one view per block, in place: views of at most ITEMS kSortThreads keys.
template <int ITEMS>
__global__ __launch_bounds__(kSortThreads) void k_sort_small(uint32_t* keys, uint32_t* vals, const uint32_t* vstart,
                                                             const unsigned long long* count, int64_t cap,
                                                             const uint32_t* overflow, int passes) {
  __shared__ uint16_t cnt[kSortWaves][kSortDigits];
  __shared__ uint32_t s_key[ITEMS * kSortThreads], s_val[ITEMS * kSortThreads];
  __shared__ uint32_t lbase[kSortDigits], red[8];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const uint32_t v0 = vstart[blockIdx.x], v1 = vstart[blockIdx.x + 1];
  const uint32_t M = clamp_count(count, cap, overflow);
  const uint32_t beg = min(v0, M);
  const uint32_t n = min(min(v1, M) - beg, uint32_t(ITEMS * kSortThreads));
  if (n <= 1) return;  // block-uniform
  // the keys past the end are all bits: they stay last, and are not written
  uint32_t key[ITEMS], val[ITEMS];
  const uint32_t first = uint32_t(w * 64 * ITEMS + lane);
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const uint32_t i = first + uint32_t(64 * r);
    key[r] = i < n ? keys[beg + i] : ~0u;
    val[r] = i < n ? vals[beg + i] : 0u;
  }
  for (int p = 0; p < passes; ++p) {
    const int shift = p * kSortBits;
    uint16_t rank[ITEMS];
    wave_rank(key, shift, cnt[w], rank);
    __syncthreads();  // (and the reads of s_key, s_val below are done)
    const uint32_t own = t < kSortDigits ? digit_offsets(cnt, t) : 0u;
    uint32_t at, unused;
    digit_scan2(own, 0u, red, at, unused);
    if (t < kSortDigits) lbase[t] = at;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const uint32_t d = (key[r] >> shift) & (kSortDigits - 1);
      const uint32_t i = lbase[d] + cnt[w][d] + rank[r];
      s_key[i] = key[r];
      s_val[i] = val[r];
    }
    __syncthreads();
    if (p + 1 == passes) break;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      key[r] = s_key[first + uint32_t(64 * r)];
      val[r] = s_val[first + uint32_t(64 * r)];
    }
  }
  for (uint32_t i = t; i < n; i += kSortThreads) {
    keys[beg + i] = s_key[i];
    vals[beg + i] = s_val[i];
  }
}

// ------------------------------------------------------------------------------------
// Device-wide exclusive scan of u32 counts, in place, in two launches: per-block sums,
// then each block adds up the sums of the blocks before it (a few hundred words at most
// for the counts of a step, read once per block) and scans its kScanTile elements from
// there; the block holding the last element writes the total.  The element count is read
// from the device (clamped to the capacity the grid was sized for) when `count` is given;
// blocks past it leave at once.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ int64_t scan_len(int64_t cap, const unsigned long long* count) {
  if (!count) return cap;
  const unsigned long long c = *count;
  return c < (unsigned long long)cap ? int64_t(c) : cap;
}

// A thread's sixteen consecutive elements from `base`, zero past n: all loads in flight at once
// (a few at a time, the sums of 640x480 with 500k Gaussians took 5.9 us a launch, now 4.6; over
// sixteen 1752x1168 views 8.3 and 5.1).
__device__ __forceinline__ void scan_load(const uint32_t* a, int64_t base, int64_t n, uint32_t (&x)[16]) {
  static_assert(kScanTile == 256 * 16, "sixteen elements a thread");
  if (base + 16 <= n) {
    const uint4* src = reinterpret_cast<const uint4*>(a + base);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint4 q = src[j];
      x[4 * j] = q.x;
      x[4 * j + 1] = q.y;
      x[4 * j + 2] = q.z;
      x[4 * j + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) x[j] = base + j < n ? a[base + j] : 0u;
  }
}

__global__ __launch_bounds__(256) void k_scan_reduce(const uint32_t* a, int64_t cap, const unsigned long long* count,
                                                     uint32_t* part) {
  __shared__ uint32_t red[4];
  const int64_t n = scan_len(cap, count);
  uint32_t x[16], sum = 0;
  scan_load(a, int64_t(blockIdx.x) * kScanTile + int64_t(threadIdx.x) * 16, n, x);
#pragma unroll
  for (int j = 0; j < 16; ++j) sum += x[j];
  const uint32_t tot = block_sum_u32(sum, red);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_scan_down(uint32_t* a, int64_t cap, const unsigned long long* count,
                                                   const uint32_t* part, unsigned long long* total) {
  __shared__ uint32_t red[4];
  const int64_t n = scan_len(cap, count);
  const int64_t b0 = int64_t(blockIdx.x) * kScanTile;
  if (b0 >= n) {  // block-uniform
    if (blockIdx.x == 0 && threadIdx.x == 0) *total = 0ull;
    return;
  }
  const int64_t base = b0 + int64_t(threadIdx.x) * 16;
  uint32_t x[16];
  scan_load(a, base, n, x);
  uint32_t before = 0;  // the sums of the blocks in front
  for (int i = int(threadIdx.x); i < int(blockIdx.x); i += 256) before += part[i];
  before = block_sum_u32(before, red);
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) sum += x[j];
  const uint32_t ex = block_exclusive_scan_u32(sum, red);
  if (threadIdx.x == 255 && b0 + kScanTile >= n) *total = (unsigned long long)before + ex + sum;
  uint32_t run = before + ex;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint32_t v = x[j];
    x[j] = run;
    run += v;
  }
  if (base + 16 <= n) {
    uint4* dst = reinterpret_cast<uint4*>(a + base);
#pragma unroll
    for (int j = 0; j < 4; ++j) dst[j] = make_uint4(x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]);
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (base + j < n) a[base + j] = x[j];
  }
}

// ------------------------------------------------------------------------------------
// K3/K4 binning (see BinPlan).  Both stages place items that cover a contiguous run of
// bins [lo, hi] (tile rows of a record, tile columns of a row entry) stably: chunk by
// chunk from scanned per-(bin, chunk) counts, and inside a chunk by one block, 256 items
// a round (place_round).
//
// A round's pairs are written densely.  Each wavefront's 64 items become one 64-bit
// coverage mask per bin (a run as two flipped bits, at lo and past hi, and an XOR scan over
// the bins); population counts give every bin's pairs and a scan their places in bin order.
// The lanes then take a bin each and list its items into LDS (as many steps as the fullest
// bin has items), and consecutive lanes write out consecutive pairs: a bin's pairs of the
// round are one contiguous run of the output.  (One bin a step for a wavefront's 64 items, the
// covering lanes storing directly, left most lanes of a store idle; and with the records of
// sixteen views interleaved every wavefront walked the rows of all of them.)
//
// Kernel trace, rows + tiles stage, that walk against this: 25 + 16 -> 23 + 16 us (640x480,
// 500k), 30 + 351 -> 23 + 168 us (1752x1168, 70M pairs), 395 + 368 -> 140 + 183 us (eight uneven
// views), 4193 + 1934 -> 867 + 783 us (sixteen 1752x1168 views).  It is bound by VALU issue
// (87 of 168 us) and by the rounds' barriers.
// ------------------------------------------------------------------------------------
constexpr int kPlaceThreads = 256;  // items of a round
constexpr int kPlaceBins = 256;     // bins handled at once (more: window after window)
constexpr int kPlaceStage = 4096;   // pairs listed at once

// The block's LDS, sized for the bins of a launch (place_lds bytes of dynamic LDS): a short one
// lets more blocks share a CU.
struct PlaceLds {
  unsigned long long* mask;  // [4][bins + 1] per wavefront and bin, the items that cover it
  uint32_t* next;   // [bins] each bin's next free slot
  uint32_t* pre;    // [bins] the round's pairs in front of each bin
  uint32_t* woff;   // [bins] within a bin, the pairs of wavefronts 0, 0-1, 0-2 (8 bits each, from bit 8)
  uint32_t* delta;  // [bins] next - pre
  uint16_t* stage;  // [kPlaceStage] (bin << 8) | item
  uint32_t* red;    // [5]: block sums, the round's pairs
  int bins;
};
static size_t place_lds(int bins) { return size_t(bins + 1) * 32 + size_t(bins) * 16 + kPlaceStage * 2 + 32; }
__device__ __forceinline__ PlaceLds place_carve(unsigned char* base, int bins) {
  PlaceLds L;
  L.bins = bins;
  L.mask = reinterpret_cast<unsigned long long*>(base);
  L.next = reinterpret_cast<uint32_t*>(base + size_t(bins + 1) * 32);
  L.pre = L.next + bins;
  L.woff = L.pre + bins;
  L.delta = L.woff + bins;
  L.red = L.delta + bins;
  L.stage = reinterpret_cast<uint16_t*>(L.red + 8);
  return L;
}

// Inclusive XOR scan over the wavefront (DPP row shifts, then the rows' totals broadcast to
// the rows behind).  Needs every lane active.
__device__ __forceinline__ uint32_t wave_xor_scan(uint32_t v) {
#define GSR_XOR_STEP(CTRL, ROWS) \
  v ^= uint32_t(__builtin_amdgcn_update_dpp(0, int(v), CTRL, ROWS, 0xF, false))
  GSR_XOR_STEP(0x111, 0xF);  // row_shr:1
  GSR_XOR_STEP(0x112, 0xF);
  GSR_XOR_STEP(0x114, 0xF);
  GSR_XOR_STEP(0x118, 0xF);
  GSR_XOR_STEP(0x142, 0xA);  // row_bcast:15
  GSR_XOR_STEP(0x143, 0xC);  // row_bcast:31
#undef GSR_XOR_STEP
  return v;
}

// Lists a wavefront's pairs of one window: lane x's bin, its items in order from place pos
// (CHECK: only places below kPlaceStage).  One item of every lane's bin a step.
template <bool CHECK>
__device__ __forceinline__ void list_items(uint16_t* stage, uint32_t m, uint32_t& pos, uint32_t code) {
  while (m) {
    if (!CHECK || pos < uint32_t(kPlaceStage)) stage[pos] = uint16_t(code + uint32_t(__builtin_ctz(m)));
    ++pos;
    m &= m - 1u;
  }
}

// One round: this thread's item covers bins [lo, hi] of nb <= L.bins (lo > hi: none); emit(slot,
// item, bin) writes a pair.  Called by all 256 threads; L.next must be ready (a barrier
// after it was written) and is advanced; ends with a barrier.
template <class Emit>
__device__ __forceinline__ void place_round(const PlaceLds& L, int nb, int lo, int hi, Emit&& emit) {
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int stride = L.bins + 1;
  unsigned long long* mask = L.mask + w * stride;
  for (int x = lane; x <= nb; x += 64) mask[x] = 0ull;
  wave_lds_sync();
  if (lo <= hi) {
    atomicXor(&mask[lo], 1ull << lane);
    atomicXor(&mask[hi + 1], 1ull << lane);
  }
  wave_lds_sync();
  unsigned long long carry = 0;
  for (int x0 = 0; x0 < nb; x0 += 64) {
    const unsigned long long v = x0 + lane < nb ? mask[x0 + lane] : 0ull;
    const uint32_t l = wave_xor_scan(uint32_t(v)), h = wave_xor_scan(uint32_t(v >> 32));
    const unsigned long long m = ((static_cast<unsigned long long>(h) << 32) | l) ^ carry;
    if (x0 + lane < nb) mask[x0 + lane] = m;
    carry ^= (static_cast<unsigned long long>(uint32_t(__builtin_amdgcn_readlane(int(h), 63))) << 32) |
             uint32_t(__builtin_amdgcn_readlane(int(l), 63));
  }
  __syncthreads();
  uint32_t tot = 0;
  if (t < nb) {
    const uint32_t c0 = __popcll(L.mask[t]), c1 = __popcll(L.mask[stride + t]), c2 = __popcll(L.mask[2 * stride + t]);
    tot = c0 + c1 + c2 + __popcll(L.mask[3 * stride + t]);
    L.woff[t] = (c0 << 8) | ((c0 + c1) << 16) | ((c0 + c1 + c2) << 24);
  }
  const uint32_t ex = block_exclusive_scan_u32(tot, L.red);
  if (t < nb) {
    const uint32_t nx = L.next[t];
    L.pre[t] = ex;
    L.delta[t] = nx - ex;
    L.next[t] = nx + tot;
  }
  if (t == kPlaceThreads - 1) L.red[4] = ex + tot;
  __syncthreads();
  const uint32_t total = L.red[4];
  for (uint32_t p0 = 0; p0 < total; p0 += kPlaceStage) {
    for (int x = lane; x < nb; x += 64) {
      const unsigned long long m = mask[x];
      uint32_t pos = L.pre[x] + (w == 0 ? 0u : (L.woff[x] >> (8 * w)) & 255u) - p0;  // (wraps in front of p0)
      const uint32_t code = (uint32_t(x) << 8) | uint32_t(64 * w);
      if (total <= uint32_t(kPlaceStage)) {
        list_items<false>(L.stage, uint32_t(m), pos, code);
        list_items<false>(L.stage, uint32_t(m >> 32), pos, code + 32u);
      } else {
        list_items<true>(L.stage, uint32_t(m), pos, code);
        list_items<true>(L.stage, uint32_t(m >> 32), pos, code + 32u);
      }
    }
    __syncthreads();
    const uint32_t n = min(total - p0, uint32_t(kPlaceStage));
    for (uint32_t i = t; i < n; i += kPlaceThreads) {
      const uint32_t code = L.stage[i];
      const uint32_t x = code >> 8;
      emit(L.delta[x] + p0 + i, int(code & 255u), int(x));
    }
    __syncthreads();
  }
}

__device__ __forceinline__ int view_of_tile(const ViewTable& vt, int tile) {
  int v = 0;
  for (int i = 1; i < vt.nviews; ++i)
    if (tile >= vt.v[i].tile_off) v = i;
  return v;
}

__device__ __forceinline__ int view_of_row(const ViewTable& vt, uint32_t row) {
  int v = 0;
  for (int i = 1; i < vt.nviews; ++i)
    if (int(row) >= vt.v[i].row_off) v = i;
  return v;
}

__device__ __forceinline__ uint32_t view_of_record(const ViewTable& vt, uint32_t rid, int64_t n) {
  return vt.nviews == 1 ? 0u : rid / uint32_t(n);
}

// The column runs that the projection kept for a record's first kRowRuns tile rows (exact tiles).
__device__ __forceinline__ void load_row_runs(const Records& rec, uint2 entry, bool valid, uint32_t (&rr)[kRowRuns]) {
#pragma unroll
  for (int j = 0; j < kRowRuns; ++j) rr[j] = 0u;
  if (!rec.runs || !valid) return;
  const uint4* src = reinterpret_cast<const uint4*>(rec.runs + int64_t(entry.x) * kRowRuns);
#pragma unroll
  for (int j = 0; j < kRowRuns / 4; ++j) {
    const uint4 q = src[j];
    rr[4 * j] = q.x;
    rr[4 * j + 1] = q.y;
    rr[4 * j + 2] = q.z;
    rr[4 * j + 3] = q.w;
  }
}

// stage 1 counts: tile-row histogram of one chunk of depth-sorted records
__global__ __launch_bounds__(256) void k_bin_rows_count(ViewTable vt, int64_t n, Records rec, const uint32_t* dvals,
                                                        const unsigned long long* nvis, int64_t cap_vis,
                                                        const uint32_t* overflow, BinPlan plan) {
  extern __shared__ uint32_t hist[];
  const int R = plan.rows;
  const int chunk = xcd_block(blockIdx.x, gridDim.x);
  if (chunk >= plan.nch1) return;  // block-uniform
  for (int i = threadIdx.x; i < R; i += 256) hist[i] = 0;
  __syncthreads();
  if (chunk == 0)  // the tile order's counters (see tile_order_count)
    for (int i = threadIdx.x; i < kOrderWords; i += 256) plan.ord[i] = 0u;
  const int64_t NV = clamp_count(nvis, cap_vis, overflow);
  const int64_t beg = int64_t(chunk) * kPlaceThreads * plan.rounds1;
  const int64_t end = min(NV, beg + int64_t(kPlaceThreads) * plan.rounds1);
  for (int64_t i = beg + threadIdx.x; i < end; i += 256) {
    const uint32_t rid = dvals[i];
    const uint2 rc = rec.rect[rid];
    const int ro = vt.v[view_of_record(vt, rid, n)].row_off;
    const int y0 = ro + int(rc.y & 0xFFFFu), y1 = min(ro + int(rc.y >> 16), R - 1);
    for (int y = y0; y <= y1; ++y) atomicAdd(&hist[y], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < R; i += 256) plan.cnt1[int64_t(i) * plan.nch1 + chunk] = hist[i];
}

// Per row: list start and length, its segments and its first flat (tile, segment) index;
// totals of segments and of the flat array.  Run by the whole of one block of NT threads
// (the last block of the row placement, before its own work: no launch of its own).
template <int NT>
__device__ void rows_meta(const ViewTable& vt, const BinPlan& plan, uint32_t* overflow, unsigned long long* part) {
  const int R = plan.rows, t = threadIdx.x;
  const int per = (R + NT - 1) / NT;
  const int beg = min(R, t * per), end = min(R, beg + per);
  const unsigned long long E1 = plan.words[0];
  const uint32_t S2 = uint32_t(kPlaceThreads) * uint32_t(plan.rounds2);
  auto row = [&](int r, uint32_t& start, uint32_t& len, uint32_t& nseg, uint32_t& w) {
    start = plan.cnt1[int64_t(r) * plan.nch1];
    const unsigned long long next = r + 1 < R ? plan.cnt1[int64_t(r + 1) * plan.nch1] : E1;
    len = uint32_t(next - start);
    nseg = (len + S2 - 1) / S2;
    w = nseg * uint32_t(vt.v[view_of_row(vt, uint32_t(r))].tiles_x);
  };
  unsigned long long sseg = 0, sw = 0;
  for (int r = beg; r < end; ++r) {
    uint32_t a, l, ns, w;
    row(r, a, l, ns, w);
    sseg += ns;
    sw += w;
  }
  const unsigned long long iseg = block_inclusive_scan_u64<NT>(sseg, part);
  __syncthreads();
  const unsigned long long iw = block_inclusive_scan_u64<NT>(sw, part);
  unsigned long long seg = iseg - sseg, flat = iw - sw;
  for (int r = beg; r < end; ++r) {
    uint32_t a, l, ns, w;
    row(r, a, l, ns, w);
    plan.rowinfo[r] = make_uint4(a, l, uint32_t(seg), uint32_t(flat));
    plan.seg_start[r] = uint32_t(seg);
    seg += ns;
    flat += w;
  }
  if (t == NT - 1) {
    const bool over = iseg > (unsigned long long)plan.cap_seg || iw > (unsigned long long)plan.cap_flat;
    if (over) raise_overflow(overflow);
    plan.seg_start[R] = uint32_t(over ? 0ull : iseg);
    plan.words[1] = over ? 0ull : iseg;
    plan.words[2] = over ? 0ull : iw;
  }
}

// stage 1 placement: one block per chunk writes (record, column run) entries into the row
// lists.  With exact tiles an entry carries the run that the projection kept for the k-th tile
// row of its record (k < kRowRuns), and past those rows the rectangle's columns marked
// kRunUncut, so that stage 2 cuts them; without exact tiles the rectangle's columns.
__global__ __launch_bounds__(kPlaceThreads) void k_bin_rows_place(ViewTable vt, int64_t n, Records rec,
                                                                  const uint32_t* dvals,
                                                                  const unsigned long long* nvis, int64_t cap_vis,
                                                                  uint32_t* overflow, BinPlan plan) {
  extern __shared__ __align__(16) unsigned char s_dyn[];  // place_lds(bins) bytes, bins = min(rows, kPlaceBins)
  __shared__ union {
    uint32_t rr[kRowRuns + 1][kPlaceThreads];   // the round's row runs, row k of item j at [k][j]
    unsigned long long meta[kPlaceThreads];     // rows_meta's, before the rounds
  } s;
  __shared__ uint32_t s_rid[kPlaceThreads], s_first[kPlaceThreads];
  const int t = threadIdx.x, R = plan.rows;
  const PlaceLds L = place_carve(s_dyn, min(R, kPlaceBins));
  if (blockIdx.x == gridDim.x - 1)
    rows_meta<kPlaceThreads>(vt, plan, overflow, s.meta);
  const int chunk = xcd_block(blockIdx.x, gridDim.x);
  const int64_t NV = clamp_count(nvis, cap_vis, overflow);
  const int64_t beg = int64_t(chunk) * kPlaceThreads * plan.rounds1;
  if (chunk >= plan.nch1 || beg >= NV) return;  // block-uniform
  // the records are in view order: the chunk's rows are those of its first to its last record's view
  const int64_t end = min(NV, beg + int64_t(kPlaceThreads) * plan.rounds1);
  const ViewDev& v0 = vt.v[view_of_record(vt, dvals[beg], n)];
  const ViewDev& v1 = vt.v[view_of_record(vt, dvals[end - 1], n)];
  const int y0 = v0.row_off, y1 = min(v1.row_off + v1.tiles_y, R);
  for (int w0 = y0; w0 < y1; w0 += kPlaceBins) {
    const int nb = min(kPlaceBins, y1 - w0);
    __syncthreads();
    if (t < nb) L.next[t] = plan.cnt1[int64_t(w0 + t) * plan.nch1 + chunk];
    for (int r = 0; r < plan.rounds1; ++r) {
      const int64_t i = beg + int64_t(r) * kPlaceThreads + t;
      if (i - t >= end) break;  // block-uniform
      int lo = 1, hi = 0;
      uint2 entry = make_uint2(0u, 0u);
      uint32_t first = 0;
      if (i < end) {
        const uint32_t rid = dvals[i];
        const uint2 rc = rec.rect[rid];
        const int ro = vt.v[view_of_record(vt, rid, n)].row_off;
        lo = ro + int(rc.y & 0xFFFFu);
        hi = min(ro + int(rc.y >> 16), R - 1);
        first = uint32_t(lo);
        entry = make_uint2(rid, rc.x);
        lo = max(lo, w0) - w0;
        hi = min(hi, w0 + nb - 1) - w0;
      }
      if (__syncthreads_or(lo <= hi) == 0) continue;
      if (rec.runs) {
        uint32_t rr[kRowRuns];
        load_row_runs(rec, entry, lo <= hi, rr);
#pragma unroll
        for (int k = 0; k < kRowRuns; ++k) s.rr[k][t] = rr[k];
      }
      s.rr[kRowRuns][t] = rec.runs ? entry.y | kRunUncut : entry.y;
      s_rid[t] = entry.x;
      s_first[t] = first;
      place_round(L, nb, lo, hi, [&](uint32_t dst, int j, int bin) {
        const uint32_t k = rec.runs ? min(uint32_t(w0 + bin) - s_first[j], uint32_t(kRowRuns)) : uint32_t(kRowRuns);
        if (int64_t(dst) < plan.cap_M) plan.rowlist[dst] = make_uint2(s_rid[j], s.rr[k][j]);
      });
    }
  }
}

// the row whose segments contain segment s: the last r with seg_start[r] <= s
__device__ __forceinline__ int row_of_segment(const uint32_t* seg_start, int R, uint32_t s) {
  int lo = 0, hi = R - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (seg_start[mid] <= s)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

struct Segment {
  uint32_t beg, end;   // entries of the row list
  uint32_t flat;       // flat index of (column 0, this segment)
  uint32_t nseg;       // segments of the row (stride between columns)
  int tiles_x;
  int row;             // global tile row
};

__device__ __forceinline__ Segment segment_of(const ViewTable& vt, const BinPlan& plan, uint32_t s) {
  const int r = row_of_segment(plan.seg_start, plan.rows, s);
  const uint4 info = plan.rowinfo[r];
  const uint32_t S2 = uint32_t(kPlaceThreads) * uint32_t(plan.rounds2);
  Segment g;
  const uint32_t sidx = s - info.z;
  g.nseg = (info.y + S2 - 1) / S2;
  g.beg = info.x + sidx * S2;
  g.end = min(info.x + info.y, g.beg + S2);
  g.flat = info.w + sidx;
  g.tiles_x = vt.v[view_of_row(vt, uint32_t(r))].tiles_x;
  g.row = r;
  return g;
}

// ------------------------------------------------------------------------------------
// Tile work queue.  Tiles are ordered by decreasing expected work (a counting sort on
// buckets of eight steps per octave, in one block: the order inside a bucket is
// arbitrary) and the compositing kernels run as persistent blocks that take the next tile
// from a device counter, so the heaviest tiles start first and light ones fill the tail.
// A tile's work is its longest per-pixel contributor count, which the list length does
// not predict (a pixel stops once its transmittance is spent); when a previous forward
// of the same tiles left those counts (`hint`), they are the key, else the list length.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t work_bucket(uint32_t w) {
  if (w == 0) return 0;
  const uint32_t e = 31u - uint32_t(__clz(w));
  const uint32_t m = e >= 3 ? (w >> (e - 3)) & 7u : (w << (3 - e)) & 7u;
  return 1u + 8u * e + m;
}

// The queue order of `total` tiles by their list lengths, by one whole block of NT threads (LDS:
// cnt and start of kOrderBuckets words, red of NT / 64): bucket counts, their scan heaviest
// bucket first, then each tile's slot (the order inside a bucket is arbitrary).
template <int NT>
__device__ void tile_order_block(const uint2* ranges, int total, uint32_t* order, uint32_t* cnt, uint32_t* start,
                                 uint32_t* red) {
  const int t = threadIdx.x;
  for (int b = t; b < kOrderBuckets; b += NT) cnt[b] = 0;
  __syncthreads();
  auto key = [&](int i) {
    const uint2 r = ranges[i];
    return work_bucket(r.y - r.x);
  };
  for (int i = t; i < total; i += NT) atomicAdd(&cnt[key(i)], 1u);
  __syncthreads();
  // heaviest bucket first: thread t takes positions t P .. t P + P - 1 of the descending order
  constexpr int P = (kOrderBuckets + NT - 1) / NT;
  uint32_t c[P], sum = 0;
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int bk = kOrderBuckets - 1 - (t * P + j);
    c[j] = bk >= 0 ? cnt[bk] : 0u;
    sum += c[j];
  }
  uint32_t run = block_exclusive_scan_u32(sum, red);
#pragma unroll
  for (int j = 0; j < P; ++j) {
    const int bk = kOrderBuckets - 1 - (t * P + j);
    if (bk >= 0) start[bk] = run;
    run += c[j];
  }
  __syncthreads();
  for (int i = t; i < total; i += NT) order[atomicAdd(&start[key(i)], 1u)] = uint32_t(i);
}

// The same order from a hint by many blocks, 256 tiles each, in the two kernels of the tile
// stage: the count kernel's blocks add their tiles' buckets to global counters
// (tile_order_count), the placement's blocks then know where every bucket starts and take
// places in it (tile_order_place).  ord: kOrderBuckets counters and as many cursors, zero at the
// start of the step.  (By one block, the order of 128k tiles took longer than the placement.)
// The hint is read once, its buckets kept in okey: another forward of the context, on a stream that
// the caller changed to, may be writing it, and places taken by other buckets than were counted
// would leave the queue with tiles missing and run past its end.
__device__ void tile_order_count(const uint32_t* hint, int total, uint32_t* ord, uint16_t* okey, uint32_t* cnt) {
  if (int(blockIdx.x) * 256 >= total) return;  // block-uniform
  for (int b = threadIdx.x; b < kOrderBuckets; b += 256) cnt[b] = 0;
  __syncthreads();
  for (int i = int(blockIdx.x) * 256 + int(threadIdx.x); i < total; i += int(gridDim.x) * 256) {
    const uint32_t b = work_bucket(hint[i]);
    okey[i] = uint16_t(b);
    atomicAdd(&cnt[b], 1u);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kOrderBuckets; b += 256)
    if (cnt[b]) atomicAdd(&ord[b], cnt[b]);
}

__device__ void tile_order_place(const uint16_t* okey, int total, uint32_t* ord, uint32_t* order, uint32_t* cnt,
                                 uint32_t* start, uint32_t* red) {
  if (int(blockIdx.x) * 256 >= total) return;  // block-uniform
  const int t = threadIdx.x;
  for (int b = t; b < kOrderBuckets; b += 256) cnt[b] = 0;
  __syncthreads();
  // this block's tiles of each bucket (their rank in it is kept in the loop below, so count first)
  for (int i = int(blockIdx.x) * 256 + t; i < total; i += int(gridDim.x) * 256) atomicAdd(&cnt[okey[i]], 1u);
  // heaviest bucket first: position t of the descending order is bucket kOrderBuckets - 1 - t; bucket 0,
  // the last, starts after all others
  const uint32_t c = ord[kOrderBuckets - 1 - t];
  const uint32_t ex = block_exclusive_scan_u32(c, red);  // (its barrier also completes cnt)
  {
    const int b = kOrderBuckets - 1 - t;
    start[b] = ex + (cnt[b] ? atomicAdd(&ord[kOrderBuckets + b], cnt[b]) : 0u);
    if (t == 255) start[0] = ex + c + (cnt[0] ? atomicAdd(&ord[kOrderBuckets], cnt[0]) : 0u);
  }
  static_assert(kOrderBuckets == 257, "one bucket per thread and bucket 0");
  __syncthreads();
  for (int i = int(blockIdx.x) * 256 + t; i < total; i += int(gridDim.x) * 256)
    order[atomicAdd(&start[okey[i]], 1u)] = uint32_t(i);
  __syncthreads();
}

__global__ __launch_bounds__(1024) void k_tile_order(const uint2* ranges, int total, uint32_t* order) {
  __shared__ uint32_t cnt[kOrderBuckets], start[kOrderBuckets];
  __shared__ uint32_t red[16];
  tile_order_block<1024>(ranges, total, order, cnt, start, red);
}

// stage 2 counts: tile-column histogram of one segment of a row list, one block per segment
// (each run adds +1 at its first column and -1 past its last, and a scan over the columns
// gives the counts).  With exact tiles the runs of a
// record's first kRowRuns rows arrive cut by the projection; a run marked kRunUncut (a
// later row of a tall splat) is cut here to the columns its ellipse reaches in this row
// (row_run) and written back, so the placement below sees the same run; a row the
// ellipse misses gets the empty run kRunEmpty (lo > hi).  With a work hint the blocks also
// count the tiles' order buckets.
__global__ __launch_bounds__(256) void k_bin_tiles_count(ViewTable vt, BinPlan plan, Records rec, float exact_k,
                                                         int tile, const uint32_t* hint) {
  extern __shared__ uint32_t hist[];  // max_tiles_x + 1 words
  __shared__ uint32_t s_cnt[kOrderBuckets], s_red[4], s_carry;
  const int t = threadIdx.x;
  if (hint) tile_order_count(hint, vt.total_tiles, plan.ord, plan.okey, s_cnt);
  const unsigned long long S = plan.words[1];
  for (uint32_t s = blockIdx.x; s < S; s += gridDim.x) {
    const Segment g = segment_of(vt, plan, s);
    __syncthreads();
    for (int i = t; i <= g.tiles_x; i += 256) hist[i] = 0;
    if (t == 0) s_carry = 0;
    __syncthreads();
    for (uint32_t i = g.beg + uint32_t(t); i < g.end; i += 256) {
      const uint2 e = plan.rowlist[i];
      uint32_t cx = e.y;
      if (cx & kRunUncut) {
        cx &= ~kRunUncut;
        const uint32_t rid = e.x;
        const ViewDev& cam = vt.v[view_of_row(vt, uint32_t(g.row))];
        const float4 sp = rec.r0[rid];  // centre and conic A, B
        const float cc = rec.r1[rid].x;
        int lo, hi;
        const bool any = row_run(sp.x, sp.y, sp.z, sp.w, cc, exact_k, tile, g.row - cam.row_off, cam.W, cam.H,
                                 int(cx & 0xFFFFu), int(cx >> 16), lo, hi);
        cx = any ? uint32_t(lo) | (uint32_t(hi) << 16) : kRunEmpty;
        plan.rowlist[i].y = cx;
      }
      const int x0 = int(cx & 0xFFFFu), x1 = min(int(cx >> 16), g.tiles_x - 1);
      if (x0 <= x1) {  // the run in difference form: +1 at its first column, -1 past its last
        atomicAdd(&hist[x0], 1u);
        atomicAdd(&hist[x1 + 1], 0xFFFFFFFFu);
      }
    }
    __syncthreads();
    for (int c0 = 0; c0 < g.tiles_x; c0 += 256) {  // inclusive scan over the columns, 256 at a time
      const int x = c0 + t;
      const uint32_t v = x < g.tiles_x ? hist[x] : 0u;
      const uint32_t carry = s_carry;
      const uint32_t in = block_exclusive_scan_u32(v, s_red) + v + carry;
      if (x < g.tiles_x) plan.cntF[g.flat + uint32_t(x) * g.nseg] = in;
      __syncthreads();
      if (t == 255) s_carry = in;
      __syncthreads();
    }
  }
}

// [start, end) of tile t from the flat scan; empty tiles are [0, 0)
__device__ __forceinline__ uint2 tile_range(const ViewTable& vt, const BinPlan& plan, const uint32_t* overflow,
                                            int t) {
  if (*overflow) return make_uint2(0u, 0u);  // nothing was binned
  const ViewDev& cam = vt.v[view_of_tile(vt, t)];
  const int local = t - cam.tile_off;
  const int r = cam.row_off + local / cam.tiles_x, x = local % cam.tiles_x;
  const uint4 info = plan.rowinfo[r];
  const uint32_t S2 = uint32_t(kPlaceThreads) * uint32_t(plan.rounds2);
  const uint32_t nseg = (info.y + S2 - 1) / S2;
  uint2 out = make_uint2(0u, 0u);
  if (nseg) {
    const unsigned long long F = plan.words[2];
    const uint32_t idx = info.w + uint32_t(x) * nseg;
    const uint32_t a = plan.cntF[idx];
    const uint32_t b = (unsigned long long)(idx + nseg) < F ? plan.cntF[idx + nseg] : uint32_t(plan.words[3]);
    if (b > a) out = make_uint2(a, b);
  }
  return out;
}

// stage 2 placement: one block per segment writes record ids into the tile lists; the blocks
// first write the tile ranges (grid-stride over the tiles) and, with a work hint, the tile
// queue's order
__global__ __launch_bounds__(kPlaceThreads) void k_bin_tiles_place(ViewTable vt, BinPlan plan, uint32_t* vals,
                                                                   const uint32_t* overflow, uint2* ranges,
                                                                   int hinted, uint32_t* order) {
  extern __shared__ __align__(16) unsigned char s_dyn[];  // place_lds(bins) bytes, bins = min(max_tiles_x, kPlaceBins)
  __shared__ uint32_t s_rid[kPlaceThreads];
  const int t = threadIdx.x;
  const PlaceLds L = place_carve(s_dyn, min(vt.max_tiles_x, kPlaceBins));
  if (hinted) {  // (in the stage's LDS, before the placement uses it)
    uint32_t* cnt = reinterpret_cast<uint32_t*>(L.stage);
    static_assert(kPlaceStage * 2 >= 2 * kOrderBuckets * 4, "the stage holds the counters and starts");
    tile_order_place(plan.okey, vt.total_tiles, plan.ord, order, cnt, cnt + kOrderBuckets, L.red);
  }
  for (int i = int(blockIdx.x) * kPlaceThreads + t; i < vt.total_tiles; i += int(gridDim.x) * kPlaceThreads)
    ranges[i] = tile_range(vt, plan, overflow, i);
  const unsigned long long S = plan.words[1];
  for (uint32_t s = blockIdx.x; s < S; s += gridDim.x) {
    const Segment g = segment_of(vt, plan, s);
    for (int w0 = 0; w0 < g.tiles_x; w0 += kPlaceBins) {
      const int nb = min(kPlaceBins, g.tiles_x - w0);
      if (t < nb) L.next[t] = plan.cntF[g.flat + uint32_t(w0 + t) * g.nseg];
      for (uint32_t r0 = g.beg; r0 < g.end; r0 += kPlaceThreads) {
        const uint32_t i = r0 + uint32_t(t);
        const uint2 e = i < g.end ? plan.rowlist[i] : make_uint2(0u, kRunEmpty);
        const int lo = max(int(e.y & 0xFFFFu), w0) - w0;
        const int hi = min(int(e.y >> 16), w0 + nb - 1) - w0;  // (lo > hi: a row the ellipse does not reach)
        s_rid[t] = e.x;
        __syncthreads();
        place_round(L, nb, lo, hi, [&](uint32_t dst, int j, int) {
          if (int64_t(dst) < plan.cap_M) vals[dst] = s_rid[j];
        });
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* p, uint32_t value, int64_t count) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < count) p[i] = value;
}

// The smallest Gaussian index with a NaN or infinite parameter (first[0] starts at
// UINT32_MAX; it stays there when every value is finite).  Grid-stride over the five
// arrays taken as one run of n * (14 + 3 (K - 1)) values.
__global__ __launch_bounds__(256) void k_first_nonfinite(GaussDev g, int K, uint32_t* first) {
  const int64_t n = g.n;
  const int64_t sizes[5] = {3 * n, 3 * n, 4 * n, n, int64_t(3) * K * n};
  const int per[5] = {3, 3, 4, 1, 3 * K};
  const float* arrs[5] = {g.means, g.scales, g.quats, g.opac, g.sh};
  const int64_t total = sizes[0] + sizes[1] + sizes[2] + sizes[3] + sizes[4];
  for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < total; i += int64_t(gridDim.x) * 256) {
    int64_t j = i;
    int a = 0;
    while (j >= sizes[a]) j -= sizes[a++];
    if (!isfinite(arrs[a][j])) atomicMin(first, uint32_t(j / per[a]));
  }
}

// Wave priority 0..3 (s_setprio takes an immediate).
__device__ __forceinline__ void set_wave_prio(int p) {
  if (p >= 3)
    __builtin_amdgcn_s_setprio(3);
  else if (p == 2)
    __builtin_amdgcn_s_setprio(2);
  else if (p == 1)
    __builtin_amdgcn_s_setprio(1);
  else
    __builtin_amdgcn_s_setprio(0);
}

// Priority of a queue position: the first sixteenth of the items (the heaviest) 3, the
// rest of the first eighth 2, of the first quarter 1, else 0.
__device__ __forceinline__ int queue_prio(int item, int total) {
  return item * 16 < total ? 3 : (item * 8 < total ? 2 : (item * 4 < total ? 1 : 0));
}

// Block-uniform: the next tile of the queue, or -1 when it is exhausted; *prio is the
// queue position's priority.
__device__ __forceinline__ int next_tile(const TileQueue& q, uint32_t* head, int total, int* s_item, int* prio) {
  __syncthreads();
  if (threadIdx.x == 0) *s_item = int(atomicAdd(head, 1u));
  __syncthreads();
  const int item = *s_item;
  *prio = item < total && q.by_work ? queue_prio(item, total) : 0;
  return item < total ? int(q.order[item]) : -1;
}

// ------------------------------------------------------------------------------------
// K6: forward compositing.  Persistent blocks take tiles from the queue; one thread per
// pixel; the tile's sorted list is staged through LDS BATCH records at a time; a tile is
// left once every pixel has reached T < T_min.
// ------------------------------------------------------------------------------------
// entries evaluated together by the forward compositing (eight ran 5% faster than four,
// sixteen another 5% faster than eight: the heaviest tiles' single-wavefront chains wait
// on one group's LDS reads and exponentials at a time)
constexpr int kFwdGroup = 16;
// list entries between two checkpoints of the forward, and so the length of a backward
// work item: 64 rather than half a batch gives the backward about twice as many items,
// so that fewer long items are left running at the end of its launch (32 was slower:
// each item has a fixed cost, its setup reads and staging, of some 10 us under load)
constexpr int kCkptStride = 64;
constexpr int kBwdGroup = 4;  // entries evaluated together by the backward compositing
static_assert(128 % kFwdGroup == 0 && kCkptStride % kFwdGroup == 0 && 128 % kCkptStride == 0,
              "batches and checkpoint strides hold whole groups");

template <int TS, int BATCH>
__global__ __launch_bounds__(TS* TS) void k_blend_fwd(ViewTable vt, Rules ru, Records rec, const uint2* ranges,
                                                     const uint32_t* vals, float* T_final, uint32_t* n_contrib,
                                                     TileQueue q, Ckpt ck) {
  constexpr int NT = TS * TS;
  constexpr int CK = kCkptStride;
  __shared__ float s_mx[BATCH], s_my[BATCH];  // splat centres
  __shared__ float4 s_q[BATCH];               // a', b', c', opacity
  __shared__ float4 s_col[BATCH];             // colour, depth
  __shared__ int s_item;
  __shared__ uint32_t s_nmax;
  const int lane = threadIdx.x & 63;
  int tile_of_block = 0;
  // checkpoint k: the state in front of list entry k * CK
  auto checkpoint = [&](int k, float T, const f32x4& C) {
    if (k > ck.kmax) return;
    float* st = ck.state + (int64_t(tile_of_block) * ck.kmax + (k - 1)) * (5 * NT) + threadIdx.x;
    st[0] = T;
    st[NT] = C[0];
    st[2 * NT] = C[1];
    st[3 * NT] = C[2];
    st[4 * NT] = C[3];
  };
  for (;;) {
    int qprio;
    const int tile = next_tile(q, q.ctrl + kHeadFwd, vt.total_tiles, &s_item, &qprio);
    if (tile < 0) return;
    tile_of_block = tile;
    if (threadIdx.x == 0) s_nmax = 0;
    const ViewDev& cam = vt.v[view_of_tile(vt, tile)];
    const int lt = tile - cam.tile_off;
    const int ty = lt / cam.tiles_x, tx = lt - ty * cam.tiles_x;
    const int px = tx * TS + int(threadIdx.x % TS), py = ty * TS + int(threadIdx.x / TS);
    const bool inside = px < cam.W && py < cam.H;
    const uint2 rg = ranges[tile];
    const int n = int(rg.y - rg.x);
    const float fpx = float(px), fpy = float(py);
    const f32x4 px4 = {fpx, fpx, fpx, fpx}, py4 = {fpy, fpy, fpy, fpy};
    float T = 1.f;
    f32x4 C = {0.f, 0.f, 0.f, 0.f};  // colour, depth
    uint32_t last = 0;
    bool done = !inside;
    // the heaviest tiles (first in the queue) bound the kernel's duration: their
    // wavefronts take issue priority from the start; any tile still running after
    // several batches is raised too
    set_wave_prio(qprio);
    for (int b0 = 0; b0 < n; b0 += BATCH) {
      if (__syncthreads_count(!done) == 0) break;
      if (b0 > 0 && b0 <= 3 * BATCH && b0 % BATCH == 0) set_wave_prio(max(qprio, b0 / BATCH));
      if (b0 > 0) checkpoint(b0 / CK, T, C);
      const int cnt = min(BATCH, n - b0);
      // a partial batch is padded to a multiple of kFwdGroup with splats of opacity -1,
      // whose alpha (-1) is below any skip threshold (which is >= 0): no pixel takes them
      for (int j = threadIdx.x; j < ((cnt + kFwdGroup - 1) & ~(kFwdGroup - 1)); j += NT) {
        float mx = 0.f, my = 0.f;
        float4 sq = make_float4(0.f, 0.f, 0.f, -1.f), sc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (j < cnt) stage_record(rec, vals[rg.x + b0 + j], mx, my, sq, sc);
        s_mx[j] = mx;
        s_my[j] = my;
        s_q[j] = sq;
        s_col[j] = sc;
      }
      __syncthreads();
      // kFwdGroup staged entries at a time: their splat values do not depend on the
      // running transmittance, so they are evaluated together (LDS reads and exponentials
      // overlap); compositing then runs in list order, straight-line: a lane that has
      // stopped (its T is below T_min), or for which the splat is below the skip
      // threshold, takes alpha 0, which adds exact zeros and keeps T.  The wavefront
      // leaves the batch once all its lanes have stopped.
      //
      // The kernel is bound by VALU issue (89% of its time over sixteen 1752x1168 views)
      // with the LDS pipe 75% busy beside it, so everything that is a product of one
      // per-entry and one per-pixel value runs as a rank-1 update on the matrix cores:
      // the offsets of four entries in one slot each for x and y (with the centres read
      // one per lane, not broadcast), and an entry's colour and depth sums in one slot
      // instead of four: 23.3 -> 16.9 issue slots and 3 -> 1.2 LDS reads per entry, 8.4 ->
      // 7.0 ms over those views, 511 -> 427 us over eight uneven views, 70 -> 60 us on one
      // 640x480 view of 500k Gaussians (images bit for bit the same).
      for (int j = 0; j < cnt; j += kFwdGroup) {
        if (__ballot(!done) == 0ull) break;
        if (j > 0 && j % CK == 0) checkpoint((b0 + j) / CK, T, C);
        const float gx = s_mx[j + (lane & (kFwdGroup - 1))], gy = s_my[j + (lane & (kFwdGroup - 1))];
        const float gc = reinterpret_cast<const float*>(s_col + j)[lane];  // lane 4 u + i: channel i of entry u
        float a[kFwdGroup];
#pragma unroll
        for (int m = 0; m < kFwdGroup / 4; ++m) {
          const f32x4 dx = mfma_rank1(gx, -1.f, px4, m), dy = mfma_rank1(gy, -1.f, py4, m);  // pixel - centre
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float4 sq = s_q[j + 4 * m + i];
            float G;
            a[4 * m + i] = splat_alpha(dx[i], dy[i], sq.x, sq.y, sq.z, sq.w, G);
          }
        }
        uint32_t lg = 0;  // 1 + the group position of the group's last contributor, 0: none
#pragma unroll
        for (int u = 0; u < kFwdGroup; ++u) {
          const bool act = !(a[u] < ru.amin) && !(T < ru.Tmin) && inside;
          const float al = act ? fminf(a[u], ru.amax) : 0.f;
          C = mfma_rank1(gc, al * T, C, u);
          T = T * (1.f - al);
          lg = act ? uint32_t(u + 1) : lg;
        }
        last = lg ? uint32_t(b0 + j) + lg : last;
        done = !inside || T < ru.Tmin;
      }
    }
    if (inside) {
      const int64_t P = int64_t(cam.W) * cam.H;
      const int64_t pix = int64_t(py) * cam.W + px;
      cam.color[pix] = C[0] + T * ru.bg[0];
      cam.color[P + pix] = C[1] + T * ru.bg[1];
      cam.color[2 * P + pix] = C[2] + T * ru.bg[2];
      if (cam.depth) cam.depth[pix] = !ru.norm_depth ? C[3] : (T < 1.f ? C[3] / (1.f - T) : 0.f);
      if (cam.alpha) cam.alpha[pix] = 1.f - T;
      T_final[cam.pix_off + pix] = T;
      n_contrib[cam.pix_off + pix] = last;
      ck.acc[cam.pix_off + pix] = make_float4(C[0], C[1], C[2], C[3]);
    }
    const uint32_t wl = wave_max_u32(last);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) atomicMax(&s_nmax, wl);
    __syncthreads();
    if (threadIdx.x == 0) {
      ck.tile_nmax[tile] = s_nmax;
      if (ck.tile_hint) ck.tile_hint[tile] = s_nmax;
    }
  }
}

// Per pixel, the list entries in front of its last contributor that passed the skip rule
// (a statistic of the forward, for inspection): the forward's alpha of each entry
// (the same staged values and splat evaluation) compared with the threshold.
__global__ __launch_bounds__(256) void k_count_used(ViewTable vt, Rules ru, Records rec, const uint2* ranges,
                                                   const uint32_t* vals, const uint32_t* n_contrib, int tile,
                                                   int64_t total_pix, uint32_t* n_used) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= total_pix) return;
  int v = 0;
  for (int k = 1; k < vt.nviews; ++k)
    if (i >= vt.v[k].pix_off) v = k;
  const ViewDev& cam = vt.v[v];
  const int64_t pix = i - cam.pix_off;
  const int py = int(pix / cam.W), px = int(pix - int64_t(py) * cam.W);
  const uint2 rg = ranges[cam.tile_off + (py / tile) * cam.tiles_x + px / tile];
  const uint32_t nc = n_contrib[i];
  const float fpx = float(px), fpy = float(py);
  uint32_t used = 0;
  for (uint32_t j = 0; j < nc && rg.x + j < rg.y; ++j) {
    float mx, my, G;
    float4 sq, col;
    stage_record(rec, vals[rg.x + j], mx, my, sq, col);
    const float a = splat_alpha(fpx - mx, fpy - my, sq.x, sq.y, sq.z, sq.w, G);
    used += !(a < ru.amin) ? 1u : 0u;
  }
  n_used[i] = used;
}

// ------------------------------------------------------------------------------------
// Backward work items, in the tile queue's longest-first order: (tile, k) for every
// checkpoint stride k that holds a contributor of some pixel of the tile, up to the
// tile's last checkpoint; one more item (tile, kmax) covers all later entries.  A block of 256
// threads lists the 256 tiles of the queue from place 256 * slice: blocks of k_bwd_items, or in a
// captured step the first blocks of the loss kernel.  Up to kListExact tiles every block adds up
// the items in front of its slice itself; beyond, k_items_sum has added up each slice (a
// block that reserved its places with an atomic instead got them in random order, and without
// the longest-first order the backward over eight 876x584 views took 955 to 1213 us, with it 921).
// One block for all 128k tiles of sixteen 1752x1168 views made the captured loss take 1252 us,
// now 308 and 5 for the sums (eight views of 876x584: 147 -> 54 and 5, one of 640x480: 12 -> 9.6); one
// reservation per tile by the forward slowed that by a fifth over eight views.
constexpr int kListExact = 4096;

__device__ __forceinline__ uint32_t tile_items(const uint32_t* order, int i, int stride, const Ckpt& ck, uint32_t& t) {
  t = order[i];
  const uint32_t nb = (ck.tile_nmax[t] + uint32_t(stride) - 1u) / uint32_t(stride);
  return nb <= uint32_t(ck.kmax) ? nb : uint32_t(ck.kmax) + 1u;
}

__global__ __launch_bounds__(256) void k_items_sum(const uint32_t* order, int total, int stride, Ckpt ck) {
  __shared__ uint32_t red[4];
  const int i = int(blockIdx.x * 256u + threadIdx.x);
  uint32_t tile;
  const uint32_t sum = block_sum_u32(i < total ? tile_items(order, i, stride, ck, tile) : 0u, red);
  if (threadIdx.x == 0) ck.slice_items[blockIdx.x] = sum;
}

__device__ void list_bwd_items(int slice, const uint32_t* order, int total, int stride, const Ckpt& ck, uint32_t* ctrl,
                               uint32_t* red) {
  const int t = threadIdx.x, i = 256 * slice + t;
  uint32_t tile = 0, u;
  const uint32_t ni = i < total ? tile_items(order, i, stride, ck, tile) : 0u;
  uint32_t before = 0;
  if (total <= kListExact) {
    for (int k = t; k < 256 * slice; k += 256) before += tile_items(order, k, stride, ck, u);
  } else {
    for (int k = t; k < slice; k += 256) before += ck.slice_items[k];
  }
  before = block_sum_u32(before, red);
  const uint32_t at = before + block_exclusive_scan_u32(ni, red);
  if (t == 255 && i + 1 >= total)  // the last slice
    ctrl[kItems] = uint32_t(min<int64_t>(int64_t(at) + ni, ck.cap_items));
  for (uint32_t k = 0; k < ni; ++k)
    if (int64_t(at) + k < ck.cap_items) ck.items[at + k] = make_uint2(tile, k);
}

__global__ __launch_bounds__(256) void k_bwd_items(const uint32_t* order, int total, int stride, Ckpt ck,
                                                  uint32_t* ctrl) {
  __shared__ uint32_t red[4];
  list_bwd_items(int(blockIdx.x), order, total, stride, ck, ctrl, red);
}

// ------------------------------------------------------------------------------------
// K7: L1 loss and its gradient with respect to the rendered colour and depth
// ------------------------------------------------------------------------------------
// host_flag (a captured step's, else null): the host's pinned copy of the sticky overflow word, which
// nothing after the forward raises.  With order non-null (a captured step) the first blocks also list the
// backward's work items (list_bwd_items) for the tiles the forward just composited.
__global__ __launch_bounds__(256) void k_loss_l1(ViewTable vt, float depth_w, float* partial, const uint32_t* order,
                                                int total_tiles, int stride, Ckpt ck, uint32_t* ctrl, uint32_t* host_flag) {
  __shared__ float red[4];
  __shared__ uint32_t ired[4];
  const ViewDev& cam = vt.v[blockIdx.y];
  if (host_flag && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
    __hip_atomic_store(host_flag, ctrl[kOverflowSticky], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (order)  // (block-uniform; more slices than blocks where tiles are few pixels)
    for (int b = int(blockIdx.y * gridDim.x + blockIdx.x); b * 256 < total_tiles; b += int(gridDim.x * gridDim.y)) {
      list_bwd_items(b, order, total_tiles, stride, ck, ctrl, ired);
      __syncthreads();
    }
  const int64_t P = int64_t(cam.W) * cam.H;
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  float part = 0.f;
  if (i < P) {
    const float inv3p = 1.f / float(3 * P), invp = 1.f / float(P);
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
      const float d = cam.color[ch * P + i] - cam.t_color[ch * P + i];
      part += fabsf(d) * inv3p;
      cam.lg_color[ch * P + i] = (d > 0.f ? inv3p : (d < 0.f ? -inv3p : 0.f));
    }
    float gd = 0.f;
    if (cam.t_depth) {
      const float td = cam.t_depth[i];
      if (td > 0.f) {
        const float d = cam.depth[i] - td;
        part += depth_w * fabsf(d) * invp;
        gd = d > 0.f ? depth_w * invp : (d < 0.f ? -depth_w * invp : 0.f);
      }
    }
    if (cam.lg_depth) cam.lg_depth[i] = gd;
  }
  for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = part;
  __syncthreads();
  if (threadIdx.x == 0) partial[int64_t(blockIdx.y) * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// the loss: the block partial sums added in a fixed order (deterministic) by one whole
// block of 256 threads (the eager sum below; in a captured step the first block of the
// backward projection), so both give the same bits
__device__ __forceinline__ void sum_loss_partials(const float* part, int count, float* loss, float* red) {
  float v = 0.f;
  for (int i = threadIdx.x; i < count; i += 256) v += part[i];
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) *loss = (red[0] + red[1]) + (red[2] + red[3]);
}

__global__ __launch_bounds__(256) void k_loss_sum(const float* part, int count, float* loss) {
  __shared__ float red[4];
  sum_loss_partials(part, count, loss, red);
}

// ------------------------------------------------------------------------------------
// K8: backward compositing, back to front over each pixel's contributors; the
// transmittance before contributor i is T_{i+1} / (1 - alpha_i), and the colour/depth
// behind i is carried as a running blend.  The work is cut into (tile, stride) items that
// run independently: an item starts from the pixel's final state when its list ends in
// the item, else from the forward's checkpoint at the item's end.  So no wavefront walks
// more than one checkpoint stride until a tile's checkpoints run out.
//
// Each wavefront walks the staged entries only down from its own longest contributor list.
// The seven per-lane partials of each splat are reduced across the wavefront to its ten
// sums (splat_sums); the wavefronts' sums meet in LDS and the block adds each splat's total
// to the 2D-gradient buffer once per item, a row at a time.

// Block-uniform: the next backward work item, or -1; the first items (the heaviest
// tiles) take a higher wave priority, as in the forward.
__device__ __forceinline__ int next_item(uint32_t* head, int total, int* s_item) {
  __syncthreads();
  if (threadIdx.x == 0) {
    // every block takes exactly one value past the end, so the taker of the last one
    // is the last to touch the head: it resets it for the next backward
    const uint32_t v = atomicAdd(head, 1u);
    *s_item = int(v);
    if (v == uint32_t(total) + gridDim.x - 1u) *head = 0u;
  }
  __syncthreads();
  const int item = *s_item;
  if (item < total) set_wave_prio(queue_prio(item, total));
  return item < total ? item : -1;
}

// K8 with PPL vertically adjacent pixels per lane: with two (tiles of 16 and 32) a
// wavefront covers 128 pixels, so each splat's partials are reduced across the
// wavefront once for twice the pixels (the pair's partials are added first); tiles of 8
// use one.  Two per lane is the build's choice for the larger tiles (kBwdPixelsPerLane);
// four ran slower on the headline view.
//
// Per pixel, back to front, with g = dL/d(colour, depth) of the pixel and B the blend of
// g . (colour, depth) of the contributors behind (B = g . (bg, 0) behind the last):
//   T_i = T_(i+1) / (1 - alpha_i),  dL/dalpha_i = T_i (g . (c_i, z_i) - B) + gA T_final / (1 - alpha_i),
//   B <- B + alpha_i (g . (c_i, z_i) - B),
// which is the per-channel recurrence of the colour behind, dotted with g once (g is fixed
// per pixel).  With w = alpha T and u = dL/da G (a = o G; zero where alpha is clamped) the
// splat's gradients are sums over the pixels: colour and depth of w g, opacity of u, and
// centre and conic of o times the offset moments of u, which the flush turns into
// gradients with the splat's conic, once per splat.
struct BwdPixel {
  float T, Tfin, gC0, gC1, gC2, gD, gATf, B, fpy;
  int top;
};

// A pixel's state at the end of work item (tile, bf): its final state when the pixel's
// list ends inside the item, else the forward's checkpoint at the item's end, with the
// colour/depth behind = (total - in front + T_final bg) / T.
template <int TS>
__device__ __forceinline__ void bwd_pixel_setup(BwdPixel& s, const ViewDev& cam, const Rules& ru, const Ckpt& ck,
                                                const float* T_final, const uint32_t* n_contrib, int tile, int bf,
                                                int lo, int hi, int px, int py, int q) {
  constexpr int NP = TS * TS;  // pixels of a tile
  const bool inside = px < cam.W && py < cam.H;
  const int64_t P = int64_t(cam.W) * cam.H;
  const int64_t pix = int64_t(py) * cam.W + px;
  s.T = 1.f;
  s.Tfin = 1.f;
  s.gC0 = s.gC1 = s.gC2 = s.gD = s.gATf = s.B = 0.f;
  s.top = 0;
  s.fpy = float(py);
  if (!inside) return;
  const int nc = int(n_contrib[cam.pix_off + pix]);
  if (nc <= lo) return;
  s.Tfin = T_final[cam.pix_off + pix];
  float gA = 0.f;
  if (cam.g_color) {
    s.gC0 = cam.g_color[pix];
    s.gC1 = cam.g_color[P + pix];
    s.gC2 = cam.g_color[2 * P + pix];
  }
  if (cam.g_depth) s.gD = cam.g_depth[pix];
  if (cam.g_alpha) gA = cam.g_alpha[pix];
  if (ru.norm_depth) {  // output Dn = D / A, A = 1 - T_final: dL/dD = g / A, dL/dA -= g Dn / A
    const float A = 1.f - s.Tfin;
    if (A > 0.f) {
      const float Dn = ck.acc[cam.pix_off + pix].w / A;
      gA -= s.gD * Dn / A;
      s.gD = s.gD / A;
    } else {
      s.gD = 0.f;
    }
  }
  s.gATf = gA * s.Tfin;
  float BC0 = ru.bg[0], BC1 = ru.bg[1], BC2 = ru.bg[2], BD = 0.f;
  if (nc <= hi) {
    s.T = s.Tfin;
    s.top = nc;
  } else {  // only single-stride items end before the list: checkpoint bf + 1 <= kmax
    const float* st = ck.state + (int64_t(tile) * ck.kmax + bf) * (5 * NP) + q;
    const float4 acc = ck.acc[cam.pix_off + pix];
    s.T = st[0];
    const float inv = 1.f / s.T;
    BC0 = (acc.x - st[NP] + s.Tfin * ru.bg[0]) * inv;
    BC1 = (acc.y - st[2 * NP] + s.Tfin * ru.bg[1]) * inv;
    BC2 = (acc.z - st[3 * NP] + s.Tfin * ru.bg[2]) * inv;
    BD = (acc.w - st[4 * NP]) * inv;
    s.top = hi;
  }
  s.B = s.gC0 * BC0 + s.gC1 * BC1 + s.gC2 * BC2 + s.gD * BD;
}

// Sums over the wavefront of a splat's seven per-lane partials, taken to the ten values of
// its gradient in 22 instructions.  q, qy, qyy are the lane's moments of u over y (offsets
// from the splat's centre), c0..c2 and z its colour and depth sums; dx is the lane's x offset,
// the same in all lanes 16 apart (a tile's columns repeat every 8 or 16 lanes).  Lane halves
// are folded pairwise (4 swaps and adds), then 16-lane rows (2); the x moments are formed on
// those column sums; then the four registers are folded into one, 8 lanes and 4 lanes apart,
// each add writing only its half's banks of four lanes (the DPP bank mask), and reduced over
// the last four.  The four lanes of bank b in row r end with value 4 r + b:
//   0 sum u, 1 u dx, 2 c1, 3 u dx^2 | 4 u dy^2, 6 z | 8 u dy, 9 u dx dy, 10 c2 | 12 c0
// (the others hold nothing of use).  Needs every lane active.
constexpr int kSumU = 0, kSumUx = 1, kSumC1 = 2, kSumUxx = 3, kSumUyy = 4, kSumZ = 6, kSumUy = 8, kSumUxy = 9,
              kSumC2 = 10, kSumC0 = 12;

__device__ __forceinline__ float splat_sums(float q, float qy, float qyy, float c0, float c1, float c2, float z,
                                            float dx) {
  auto fold_halves = [](float a, float b) {  // lanes 0-31: a summed 32 apart; lanes 32-63: b
    swap_halves(a, b);
    return a + b;
  };
  auto fold_rows = [](float a, float b) {  // even rows: a summed 16 apart; odd rows: b
    swap_rows(a, b);
    return a + b;
  };
  const float r0 = fold_rows(fold_halves(q, qy), fold_halves(qyy, c0));  // rows: q, qyy, qy, c0
  const float r1 = fold_rows(fold_halves(c1, c2), fold_halves(z, z));    // rows: c1, z, c2, z
  const float r2 = r0 * dx, r3 = r2 * dx;                                // q dx, -, qy dx, - | q dx^2, -, -, -
  float f0, f1, g;
  // (a DPP operand needs two instructions between its write and its use)
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %4, %4 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %1, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "s_nop 0\n\t"
      "v_add_f32_dpp %2, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 1\n\t"
      "v_add_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_add_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
      : "=&v"(f0), "=&v"(f1), "=&v"(g)
      : "v"(r0), "v"(r1), "v"(r2), "v"(r3));
  return g;
}

// The flush of a stage's sums (s_g: sixteen slots per splat and wavefront) into the 2D-gradient
// rows.  One lane per splat adds up the wavefronts that hit it (s_hit; with eight of them, a
// pass over all threads before) and turns the moments into gradients: with the staged conic
// (a', b', c') = (A, 2B, C) (-log2 e / 2), (A dx + B dy, B dx + C dy) =
// -ln 2 (2a' dx + b' dy, b' dx + 2c' dy), so
//   dmu = -ln 2 o (2a' Ux + b' Uy, b' Ux + 2c' Uy),  d(A, B, C) = -o (Uxx / 2, Uxy, Uyy / 2).
// Then the values are added splat-major: consecutive lanes take consecutive values of a few
// rows, so one atomic instruction touches a few rows (cache lines), and a row's ten values
// go out together.  (Atomics are carried out at the memory side, where their number counts:
// with the centre's two values issued apart from the others the kernel took 170 us over
// one 876x584 view of a 170k map, together 130.)
template <int NT, int NW, int SB>
__device__ __forceinline__ void flush_splat_sums(float (&s_g)[NW][SB][16], const uint64_t (&s_hit)[NW],
                                                 const uint32_t* s_id, const float4* s_q, int nstage, float* grad2d) {
  constexpr float kNegLn2 = -0.69314718055994531f;
  if constexpr (NW > 2) {
    for (int i = threadIdx.x; i < 16 * nstage; i += NT) {
      const int j = i >> 4, k = i & 15;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) v += (s_hit[w] >> j) & 1ull ? s_g[w][j][k] : 0.f;
      s_g[0][j][k] = v;
    }
    __syncthreads();
  }
  for (int j = threadIdx.x; j < nstage; j += NT) {
    auto sum = [&](int k) {
      if constexpr (NW > 2) return s_g[0][j][k];
      float v = (s_hit[0] >> j) & 1ull ? s_g[0][j][k] : 0.f;
      if constexpr (NW == 2) v += (s_hit[1] >> j) & 1ull ? s_g[1][j][k] : 0.f;
      return v;
    };
    const float4 sq = s_q[j];
    const float ol = sq.w * kNegLn2, ux = sum(kSumUx), uy = sum(kSumUy);
    const float v[10] = {ol * (2.f * sq.x * ux + sq.y * uy),
                         ol * (sq.y * ux + 2.f * sq.z * uy),
                         -0.5f * sq.w * sum(kSumUxx),
                         -sq.w * sum(kSumUxy),
                         -0.5f * sq.w * sum(kSumUyy),
                         sum(kSumU),
                         sum(kSumC0),
                         sum(kSumC1),
                         sum(kSumC2),
                         sum(kSumZ)};
#pragma unroll
    for (int k = 0; k < 10; ++k) s_g[0][j][k] = v[k];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 10 * nstage; i += NT) {
    const int j = i / 10, k = i - 10 * j;
    const float v = s_g[0][j][k];
    if (v != 0.f) unsafeAtomicAdd(grad2d + int64_t(s_id[j]) * kGrad2D + k, v);
  }
}

template <int TS, int PPL>
__global__ __launch_bounds__(TS* TS / PPL) __attribute__((amdgpu_waves_per_eu(TS == 32 ? 4 : 5))) void k_blend_bwd2(
    ViewTable vt, Rules ru, Records rec, const uint2* ranges, const uint32_t* vals, const float* T_final,
    const uint32_t* n_contrib, float* grad2d, TileQueue q, Ckpt ck) {
  constexpr int NT = TS * TS / PPL;  // threads
  constexpr int NW = NT / 64;        // wavefronts
  constexpr int WX = TS < 16 ? TS : 16;  // a wavefront's pixels: WX wide, 8 high (splat_sums needs
  static_assert(64 * PPL == 8 * WX, "");  // lanes 16 apart in one column)
  constexpr int SB = kCkptStride;    // entries staged at a time: one checkpoint stride
  constexpr int GS = kBwdGroup;
  static_assert(SB % GS == 0 && GS % 4 == 0, "a stage holds whole groups, a group whole matrix operands");
  __shared__ float2 s_mu[SB];           // splat centres
  __shared__ float4 s_q[SB];            // a', b', c', opacity
  __shared__ float s_c[4][SB];          // colour, depth
  __shared__ uint32_t s_id[SB];
  __shared__ float s_g[NW][SB][16];     // per wavefront and staged splat it hit, its sums (splat_sums)
  __shared__ uint64_t s_hit[NW];        // per wavefront, the staged splats some pixel of it takes
  __shared__ uint32_t s_max;
  __shared__ int s_item;
  const int wv = int(threadIdx.x) >> 6;
  const int total = int(q.ctrl[kItems]);
  const int lane = threadIdx.x & 63;
  // this lane's pixels within the tile: column cx, rows ry .. ry + PPL - 1
  const int cx = WX * (wv % (TS / WX)) + lane % WX, ry = 8 * (wv / (TS / WX)) + PPL * (lane / WX);
  for (;;) {
    const int item = next_item(q.ctrl + kHeadBwd, total, &s_item);
    if (item < 0) return;
    const uint2 it = ck.items[item];
    const int tile = int(it.x), bf = int(it.y);
    const ViewDev& cam = vt.v[view_of_tile(vt, tile)];
    const int lt = tile - cam.tile_off;
    const int ty = lt / cam.tiles_x, tx = lt - ty * cam.tiles_x;
    const int px = tx * TS + cx, py = ty * TS + ry;
    const uint2 rg = ranges[tile];
    constexpr int CK = kCkptStride;  // checkpoint stride of the forward
    const int lo = bf * CK;        // the item's list entries: [lo, hi)
    const int hi = bf < ck.kmax ? lo + CK : int(rg.y - rg.x);
    BwdPixel p[PPL];
    int ptop = 0;
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      bwd_pixel_setup<TS>(p[i], cam, ru, ck, T_final, n_contrib, tile, bf, lo, hi, px, py + i, (ry + i) * TS + cx);
      ptop = max(ptop, p[i].top);
    }
    const int wmax = int(wave_max_u32(uint32_t(ptop)));
    if (threadIdx.x == 0) s_max = 0;
    __syncthreads();
    if (lane == 0 && wmax) atomicMax(&s_max, uint32_t(wmax));
    __syncthreads();
    const int bmax = int(s_max);
    const float fpx = float(px);
    for (int bend = bmax; bend > lo; bend -= SB) {
      const int bstart = max(lo, bend - SB);
      const int nstage = bend - bstart;
      __syncthreads();
      for (int j = threadIdx.x; j < nstage; j += NT) {
        const uint32_t id = vals[rg.x + bstart + j];
        float mx, my;
        float4 sq, sc;
        stage_record(rec, id, mx, my, sq, sc);
        s_id[j] = id;
        s_mu[j] = make_float2(mx, my);
        s_q[j] = sq;
        s_c[0][j] = sc.x;
        s_c[1][j] = sc.y;
        s_c[2][j] = sc.z;
        s_c[3][j] = sc.w;
      }
      __syncthreads();
      // Groups of staged entries, back to front.  First everything that does not depend on the
      // running T and B, for the whole group at once (its LDS reads and exponentials overlap);
      // g . (colour, depth) as rank-1 updates on the matrix cores (four entries each).  Then the
      // recurrences and sums, entry by entry; entries that no pixel of the wavefront takes are
      // left out.  A lane that does not take
      // an entry (past its list or the stage, or below the skip threshold) has alpha = 0, which
      // leaves T and B unchanged (1 / (1 - 0) = 1 exactly) and gives u = w = 0.
      //
      // The kernel is bound by VALU issue where many items are in flight, and by its items'
      // latency where few are; measured issue costs per wavefront instruction are 2 cycles for
      // adds, multiplies and fmas, 4 for compares, selects, min and DPP, 8 for exponentials,
      // reciprocals, lane swaps and the 4x4x1 products.  Against one entry at a time and centre
      // atomics of their own: 15.1 -> 12.7 ms over sixteen 1752x1168 views, 1228 -> 979 us over
      // eight uneven ones, 204 -> 145 us and 163 -> 137 us on one 876x584 (170k splats) and one
      // 640x480 view (500k).  The clamp tested at every pixel, the moments from each pixel's own
      // offset and the select of u cost 2.2% of it over many views.  Taking the sums as matrix products
      // (16x16x4, splats by pixels) was slower over many views (by a half): they share the
      // VALU's issue at 32 cycles each and need 30 KB of LDS a block.
      uint64_t hit = 0;  // staged splats some pixel of the wavefront takes (wavefront-uniform)
      for (int jb = (min(nstage, wmax - bstart) - 1) & ~(GS - 1); jb >= 0; jb -= GS) {
        const int je = jb + (lane & (GS - 1));
        const float e0 = s_c[0][je], e1 = s_c[1][je], e2 = s_c[2][je], e3 = s_c[3][je];
        float G[GS][PPL], o[GS];  // (alpha before the clamp is o G)
        bool act[GS][PPL];
        float dx[GS], dy[GS][PPL];
        f32x4 S[GS / 4][PPL];
        uint32_t hits = 0;
        int lim[PPL];  // the pixels' entries of this group
#pragma unroll
        for (int i = 0; i < PPL; ++i) {
          lim[i] = min(p[i].top, bend) - (bstart + jb);
#pragma unroll
          for (int h = 0; h < GS / 4; ++h) {
            S[h][i] = mfma_rank1(e0, p[i].gC0, f32x4{0.f, 0.f, 0.f, 0.f}, h);
            S[h][i] = mfma_rank1(e1, p[i].gC1, S[h][i], h);
            S[h][i] = mfma_rank1(e2, p[i].gC2, S[h][i], h);
            S[h][i] = mfma_rank1(e3, p[i].gD, S[h][i], h);
          }
        }
#pragma unroll
        for (int j = 0; j < GS; ++j) {
          const float4 sq = s_q[jb + j];
          const float2 mu = s_mu[jb + j];
          dx[j] = fpx - mu.x;
          o[j] = sq.w;
#pragma unroll
          for (int i = 0; i < PPL; ++i) {
            dy[j][i] = p[i].fpy - mu.y;
            const float a = splat_alpha(dx[j], dy[j][i], sq.x, sq.y, sq.z, sq.w, G[j][i]);
            act[j][i] = j < lim[i] && !(a < ru.amin);
            hits |= __ballot(act[j][i]) != 0ull ? 1u << j : 0u;
          }
        }
        hit |= uint64_t(hits) << jb;
#pragma unroll
        for (int j = GS - 1; j >= 0; --j) {
          if (!((hits >> j) & 1u)) continue;
          float u[PPL], c0 = 0.f, c1 = 0.f, c2 = 0.f, z = 0.f;
#pragma unroll
          for (int i = 0; i < PPL; ++i) {
            // The clamp is tested at every pixel: an opacity below alpha_max does not rule it out, for the
            // conic of a long thin splat comes from a det = a c - b^2 that cancels, and with it
            // q' can come out positive (G of 1.03 at the default low-pass, over 40 without one).
            const float a = o[j] * G[j][i];
            const bool below = a <= ru.amax;
            const float al = act[j][i] ? (below ? a : ru.amax) : 0.f;
            const float iom = __builtin_amdgcn_rcpf(1.f - al);
            p[i].T *= iom;
            const float w = al * p[i].T;
            const float D = S[j / 4][i][j % 4] - p[i].B;
            p[i].B += al * D;
            // (selected, not multiplied by zero: a NaN or infinity in a pixel's gradient stays with the
            // splats that the pixel takes)
            u[i] = act[j][i] && below ? (p[i].T * D + p[i].gATf * iom) * G[j][i] : 0.f;
            c0 += p[i].gC0 * w;
            c1 += p[i].gC1 * w;
            c2 += p[i].gC2 * w;
            z += p[i].gD * w;
          }
          // the lane's moments of u over y, each pixel's from its own offset (taken from the first
          // pixel's, as dy + 1, a pixel close to the splat's row leaves the rounding of larger terms)
          float q = u[0], qy = dy[j][0] * u[0], qyy = dy[j][0] * qy;
          if constexpr (PPL == 2) {
            const float y1 = dy[j][1] * u[1];
            q += u[1];
            qyy = __builtin_fmaf(dy[j][1], y1, qyy);
            qy += y1;
          }
          // (each bank of four lanes holds one of the sums: they store the same word)
          s_g[wv][jb + j][lane >> 2] = splat_sums(q, qy, qyy, c0, c1, c2, z, dx[j]);
        }
      }
      if (lane == 0) s_hit[wv] = hit;
      __syncthreads();
      flush_splat_sums<NT, NW, SB>(s_g, s_hit, s_id, s_q, nstage, grad2d);
    }
  }
}

// ------------------------------------------------------------------------------------
// K9: chain rule per Gaussian, summed over views in view order
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void store_grad(float* p, float v, int acc) {
  if (acc)
    *p += v;
  else
    *p = v;
}

// K9a: the colour term.  Four lanes per Gaussian, one per colour channel (the fourth
// idles), so a lane holds one channel's K coefficients.  Per visible view: the basis at
// the view direction, the channel's colour before the clamp, the coefficient gradient
// Y_k * dL/dc (zero where the clamp is active) and the view-direction gradient, summed
// over the channel lanes and taken through the normalisation to the mean (dp_sh).
// Coefficients pass through LDS so the [N, K, 3] loads and stores are contiguous; a
// Gaussian invisible in every view reads none and gets zero gradients.
constexpr int kShGaussians = 64;  // Gaussians per block of k_project_bwd_sh

template <int DEG>
__global__ __launch_bounds__(256) void k_project_bwd_sh(GaussDev g, ViewTable vt, Records rec, const float* grad2d,
                                                        GradOut out, float* dp_sh, AdamDev adam) {
  constexpr int K = (DEG + 1) * (DEG + 1);
  constexpr int KK = K * 3;
  constexpr bool kVec = KK % 4 == 0;  // degrees 1 and 3: whole float4s per Gaussian
  constexpr int STRIDE = KK | 1;
  __shared__ float s_sh[kShGaussians * STRIDE];
  __shared__ uint32_t s_vis[kShGaussians];
  const int t = threadIdx.x;
  const int64_t g0 = int64_t(blockIdx.x) * kShGaussians;
  const int nb = int(min<int64_t>(kShGaussians, g.n - g0));
  const int gl = t >> 2, ch = t & 3;
  const int64_t gi = g0 + gl;
  // this lane's mean and first view's colour gradient, loaded before the block stages the
  // coefficients (their latency overlaps the staging)
  float p0 = 0.f, p1 = 0.f, p2 = 0.f, dc0 = 0.f;
  uint32_t cnt0 = 0;
  if (gl < nb && ch < 3) {
    cnt0 = rec.counts[gi];
    if (cnt0) {
      p0 = g.means[gi * 3];
      p1 = g.means[gi * 3 + 1];
      p2 = g.means[gi * 3 + 2];
      dc0 = grad2d[gi * kGrad2D + 6 + ch];
    }
  }
  if (t < kShGaussians) {
    uint32_t vis = 0;
    if (t < nb)
      for (int v = 0; v < vt.nviews; ++v) vis |= rec.counts[int64_t(v) * g.n + g0 + t];
    s_vis[t] = vis;
  }
  __syncthreads();
  // 16-byte loads where the array allows them (with KK a multiple of 4 a float4 never
  // straddles two Gaussians)
  const bool vec_in = kVec && (reinterpret_cast<uintptr_t>(g.sh) & 15u) == 0;
  if (vec_in) {
    const float4* src = reinterpret_cast<const float4*>(g.sh + g0 * KK);
    for (int i = t; i < nb * (KK / 4); i += 256) {
      const int r = (4 * i) / KK, j = 4 * i - r * KK;
      const float4 v = s_vis[r] ? src[i] : make_float4(0.f, 0.f, 0.f, 0.f);
      float* d = s_sh + r * STRIDE + j;
      d[0] = v.x;
      d[1] = v.y;
      d[2] = v.z;
      d[3] = v.w;
    }
  } else {
    for (int i = t; i < nb * KK; i += 256) {
      const int r = i / KK;
      s_sh[r * STRIDE + (i - r * KK)] = s_vis[r] ? g.sh[g0 * KK + i] : 0.f;
    }
  }
  __syncthreads();
  const bool mine = gl < nb && s_vis[gl] != 0u;
  float dsh[K], dp[3] = {0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < K; ++k) dsh[k] = 0.f;
  if (mine && ch < 3) {
    float shc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) shc[k] = s_sh[gl * STRIDE + k * 3 + ch];
    if (!cnt0) {  // visible only in later views: the mean was not loaded above
      p0 = g.means[gi * 3];
      p1 = g.means[gi * 3 + 1];
      p2 = g.means[gi * 3 + 2];
    }
    for (int v = 0; v < vt.nviews; ++v) {
      const int64_t rid = int64_t(v) * g.n + gi;
      if ((v == 0 ? cnt0 : rec.counts[rid]) == 0) continue;
      const ViewDev& cam = vt.v[v];
      const float d0 = p0 - cam.cam_pos[0], d1 = p1 - cam.cam_pos[1], d2 = p2 - cam.cam_pos[2];
      const float il = 1.f / __builtin_sqrtf(d0 * d0 + d1 * d1 + d2 * d2);
      const float vx = d0 * il, vy = d1 * il, vz = d2 * il;
      float Y[K];
      sh_basis<DEG>(vx, vy, vz, Y);
      float raw = 0.5f;
#pragma unroll
      for (int k = 0; k < K; ++k) raw += shc[k] * Y[k];
      const float dc = raw > 0.f ? (v == 0 ? dc0 : grad2d[rid * kGrad2D + 6 + ch]) : 0.f;
#pragma unroll
      for (int k = 0; k < K; ++k) dsh[k] += Y[k] * dc;
      if (DEG > 0) {
        float wk[K], dv[3];
#pragma unroll
        for (int k = 0; k < K; ++k) wk[k] = shc[k] * dc;
        sh_grad_dot<DEG>(vx, vy, vz, wk, dv);
        const float vd = dv[0] * vx + dv[1] * vy + dv[2] * vz;
        dp[0] += (dv[0] - vx * vd) * il;
        dp[1] += (dv[1] - vy * vd) * il;
        dp[2] += (dv[2] - vz * vd) * il;
      }
    }
  }
  // the direction term is linear in the coefficients: sum the channel lanes (a quad)
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    dp[i] += dpp_move<0xB1, 0xF>(dp[i]);
    dp[i] += dpp_move<0x4E, 0xF>(dp[i]);
  }
  if (mine && ch == 0)
#pragma unroll
    for (int i = 0; i < 3; ++i) dp_sh[gi * 3 + i] = dp[i];
  if (!out.sh && !adam.on) return;
  __syncthreads();
  if (gl < nb && ch < 3)
#pragma unroll
    for (int k = 0; k < K; ++k) s_sh[gl * STRIDE + k * 3 + ch] = dsh[k];
  __syncthreads();
  if (adam.on) {  // one Adam step of every coefficient of the block's Gaussians, in place
    if (adam.skip && *adam.skip) return;  // the step overflowed: parameters stay as they are
    const float bc1 = adam.bc[0], bc2 = adam.bc[1];
    auto al = [](const float* q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; };
    if (kVec && al(adam.p[G_SH]) && al(adam.m[G_SH]) && al(adam.v[G_SH])) {  // 16-byte accesses
      const int64_t e0 = g0 * (KK / 4);
      for (int i = t; i < nb * (KK / 4); i += 256) {
        const int r = (4 * i) / KK, j = 4 * i - r * KK;
        const float* gs = s_sh + r * STRIDE + j;
        float4 x = reinterpret_cast<const float4*>(adam.p[G_SH])[e0 + i];
        float4 m = reinterpret_cast<const float4*>(adam.m[G_SH])[e0 + i];
        float4 v = reinterpret_cast<const float4*>(adam.v[G_SH])[e0 + i];
        auto lr = [&](int k) { return j + k < 3 ? adam.lr[G_SH] : adam.lr[G_SH + 1]; };
        x.x = adam_value<G_SH>(x.x, gs[0], m.x, v.x, lr(0), adam, bc1, bc2);
        x.y = adam_value<G_SH>(x.y, gs[1], m.y, v.y, lr(1), adam, bc1, bc2);
        x.z = adam_value<G_SH>(x.z, gs[2], m.z, v.z, lr(2), adam, bc1, bc2);
        x.w = adam_value<G_SH>(x.w, gs[3], m.w, v.w, lr(3), adam, bc1, bc2);
        reinterpret_cast<float4*>(adam.p[G_SH])[e0 + i] = x;
        reinterpret_cast<float4*>(adam.m[G_SH])[e0 + i] = m;
        reinterpret_cast<float4*>(adam.v[G_SH])[e0 + i] = v;
      }
      return;
    }
    for (int i = t; i < nb * KK; i += 256) {
      const int r = i / KK, j = i - r * KK;
      const int64_t e = g0 * KK + i;
      adam_apply<G_SH>(adam, e, adam.p[G_SH][e], s_sh[r * STRIDE + j], j < 3 ? adam.lr[G_SH] : adam.lr[G_SH + 1],
                       bc1, bc2);
    }
    return;
  }
  if (kVec && (reinterpret_cast<uintptr_t>(out.sh) & 15u) == 0 && !out.accumulate) {
    float4* dst = reinterpret_cast<float4*>(out.sh + g0 * KK);
    for (int i = t; i < nb * (KK / 4); i += 256) {
      const int r = (4 * i) / KK, j = 4 * i - r * KK;
      const float* v = s_sh + r * STRIDE + j;
      dst[i] = make_float4(v[0], v[1], v[2], v[3]);
    }
    return;
  }
  for (int i = t; i < nb * KK; i += 256) {
    const int r = i / KK;
    store_grad(out.sh + g0 * KK + i, s_sh[r * STRIDE + (i - r * KK)], out.accumulate);
  }
}

// K9b: the geometric chain rule, one thread per Gaussian; adds the colour term's
// gradient with respect to the mean (dp_sh, from K9a).
__global__ __launch_bounds__(kProjThreads) void k_project_bwd_geo(GaussDev g, ViewTable vt, Rules ru, Records rec,
                                                                  const float* grad2d, const float* dp_sh,
                                                                  GradOut out, AdamDev adam, const float* loss_part,
                                                                  int loss_np, float* loss) {
  __shared__ float lred[4];
  // a captured step adds up its loss here (block-uniform; no launch of its own)
  if (loss && blockIdx.x == 0) sum_loss_partials(loss_part, loss_np, loss, lred);
  const int64_t gi = int64_t(blockIdx.x) * kProjThreads + threadIdx.x;
  if (gi >= g.n) return;
  // the geometry is read for a Gaussian some view sees (or for the Adam step, which moves
  // every element); the others only get zero gradients
  uint32_t seen = 0;
  for (int v = 0; v < vt.nviews && !seen; ++v) seen = rec.counts[int64_t(v) * g.n + gi];
  float p[3] = {0.f, 0.f, 0.f}, s[3] = {0.f, 0.f, 0.f}, q[4] = {0.f, 0.f, 0.f, 0.f};
  if (seen || adam.on) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      p[i] = g.means[gi * 3 + i];
      s[i] = g.scales[gi * 3 + i];
    }
    const float4 q4 = reinterpret_cast<const float4*>(g.quats)[gi];
    q[0] = q4.x;
    q[1] = q4.y;
    q[2] = q4.z;
    q[3] = q4.w;
  }
  float dp[3] = {0.f, 0.f, 0.f}, ds[3] = {0.f, 0.f, 0.f}, dq[4] = {0.f, 0.f, 0.f, 0.f}, dop = 0.f;
  bool any = false;
  for (int v = 0; v < vt.nviews; ++v) {
    const int64_t rid = int64_t(v) * g.n + gi;
    if (rec.counts[rid] == 0) continue;
    any = true;
    const ViewDev& cam = vt.v[v];
    const float4* G4 = reinterpret_cast<const float4*>(grad2d + rid * kGrad2D);
    const float4 ga = G4[0], gb = G4[1], gc = G4[2];
    const float dmux = ga.x, dmuy = ga.y, dA = ga.z, dB = ga.w, dC = gb.x, dO = gb.y;
    const float dz = gc.y;
    Proj pr;
    discrete_stage(p, s, q, cam, ru.k, ru.lowpass, ru.guard, ru.jclamp, pr);
    float A, B, C;
    conic_of(pr.a, pr.b, pr.c, A, B, C);
    dop += dO;
    // conic -> projected covariance: dS = -Q G_Q Q with G_Q = [[dA, dB/2], [dB/2, dC]]
    const float hB = 0.5f * dB;
    const float QG00 = A * dA + B * hB, QG01 = A * hB + B * dC;
    const float QG10 = B * dA + C * hB, QG11 = B * hB + C * dC;
    const float S00 = -(QG00 * A + QG01 * B);
    const float S01 = -(QG00 * B + QG01 * C);
    const float S11 = -(QG10 * B + QG11 * C);
    // Sigma_hat = U U^T + lowpass I with U = T M: dU = 2 dS U
    float dU[6];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      dU[k] = 2.f * (S00 * pr.U[k] + S01 * pr.U[3 + k]);
      dU[3 + k] = 2.f * (S01 * pr.U[k] + S11 * pr.U[3 + k]);
    }
    // dT = dU M^T, dM = T^T dU
    float dT[6], dM[9];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j)
        dT[i * 3 + j] = dU[i * 3 + 0] * pr.m[j * 3 + 0] + dU[i * 3 + 1] * pr.m[j * 3 + 1] + dU[i * 3 + 2] * pr.m[j * 3 + 2];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) dM[j * 3 + k] = pr.T[j] * dU[k] + pr.T[3 + j] * dU[3 + k];
    // T = J W: dJ = dT W^T (only the four non-constant entries of J matter)
    const float* W = cam.R;
    const float dJ00 = dT[0] * W[0] + dT[1] * W[1] + dT[2] * W[2];
    const float dJ02 = dT[0] * W[6] + dT[1] * W[7] + dT[2] * W[8];
    const float dJ11 = dT[3] * W[3] + dT[4] * W[4] + dT[5] * W[5];
    const float dJ12 = dT[3] * W[6] + dT[4] * W[7] + dT[5] * W[8];
    const float tx = pr.tx, ty = pr.ty, tz = pr.tz;
    const float iz = 1.f / tz, iz2 = iz * iz, iz3 = iz2 * iz;
    const float fx = cam.fx, fy = cam.fy;
    // J02 = -fx x' / z^2 with x' = tx, or +-limit tz where clamped: d/dtx of a clamped
    // entry is 0 and its d/dtz is -J02 / tz (2 fx x' / z^3 halved); likewise J12
    const float kx = pr.clx ? 1.f : 2.f, ky = pr.cly ? 1.f : 2.f;
    const float dtx = (pr.clx ? 0.f : -fx * iz2 * dJ02) + fx * iz * dmux;
    const float dty = (pr.cly ? 0.f : -fy * iz2 * dJ12) + fy * iz * dmuy;
    const float dtz = -fx * iz2 * dJ00 + kx * fx * pr.txj * iz3 * dJ02 - fy * iz2 * dJ11 + ky * fy * pr.tyj * iz3 * dJ12 -
                      fx * tx * iz2 * dmux - fy * ty * iz2 * dmuy + dz;
#pragma unroll
    for (int j = 0; j < 3; ++j) dp[j] += W[j] * dtx + W[3 + j] * dty + W[6 + j] * dtz;
    // M = R diag(s)
    float dR[9];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        ds[j] += dM[i * 3 + j] * pr.r[i * 3 + j];
        dR[i * 3 + j] = dM[i * 3 + j] * s[j];
      }
    // R(q^) partials contracted with dR
    const float w = pr.qw, x = pr.qx, y = pr.qy, z = pr.qz;
    const float dqw = 2.f * (-z * dR[1] + y * dR[2] + z * dR[3] - x * dR[5] - y * dR[6] + x * dR[7]);
    const float dqx = 2.f * (y * dR[1] + z * dR[2] + y * dR[3] - 2.f * x * dR[4] - w * dR[5] + z * dR[6] + w * dR[7] -
                             2.f * x * dR[8]);
    const float dqy = 2.f * (-2.f * y * dR[0] + x * dR[1] + w * dR[2] + x * dR[3] + z * dR[5] - w * dR[6] + z * dR[7] -
                             2.f * y * dR[8]);
    const float dqz = 2.f * (-2.f * z * dR[0] - w * dR[1] + x * dR[2] + w * dR[3] - 2.f * z * dR[4] + y * dR[5] +
                             x * dR[6] + y * dR[7]);
    const float qd = dqw * w + dqx * x + dqy * y + dqz * z;
    const float inq = 1.f / pr.nq;
    dq[0] += (dqw - w * qd) * inq;
    dq[1] += (dqx - x * qd) * inq;
    dq[2] += (dqy - y * qd) * inq;
    dq[3] += (dqz - z * qd) * inq;
  }
  if (any) {
#pragma unroll
    for (int i = 0; i < 3; ++i) dp[i] += dp_sh[gi * 3 + i];
  }
  if (adam.on) {  // one Adam step of the Gaussian's geometry, in place
    if (adam.skip && *adam.skip) return;  // the step overflowed: parameters stay as they are
    const float bc1 = adam.bc[0], bc2 = adam.bc[1];
#pragma unroll
    for (int i = 0; i < 3; ++i) adam_apply<G_MEANS>(adam, gi * 3 + i, p[i], dp[i], adam.lr[G_MEANS], bc1, bc2);
#pragma unroll
    for (int i = 0; i < 3; ++i) adam_apply<G_SCALES>(adam, gi * 3 + i, s[i], ds[i], adam.lr[G_SCALES], bc1, bc2);
#pragma unroll
    for (int i = 0; i < 4; ++i) adam_apply<G_QUATS>(adam, gi * 4 + i, q[i], dq[i], adam.lr[G_QUATS], bc1, bc2);
    adam_apply<G_OPAC>(adam, gi, g.opac[gi], dop, adam.lr[G_OPAC], bc1, bc2);
    return;
  }
  const int acc = out.accumulate;
  if (out.means)
    for (int i = 0; i < 3; ++i) store_grad(out.means + gi * 3 + i, dp[i], acc);
  if (out.scales)
    for (int i = 0; i < 3; ++i) store_grad(out.scales + gi * 3 + i, ds[i], acc);
  if (out.quats) {
    if (!acc && (reinterpret_cast<uintptr_t>(out.quats) & 15u) == 0)
      reinterpret_cast<float4*>(out.quats)[gi] = make_float4(dq[0], dq[1], dq[2], dq[3]);
    else
      for (int i = 0; i < 4; ++i) store_grad(out.quats + gi * 4 + i, dq[i], acc);
  }
  if (out.opac) store_grad(out.opac + gi, dop, acc);
}

inline unsigned blocks_for(int64_t n, int per) { return unsigned((n + per - 1) / per); }

}  // namespace

// ------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------
hipError_t launch_project(int deg, const GaussDev& g, const ViewTable& vt, const Rules& ru, int tile,
                          const Records& rec, uint2* blocksums, int nblk, float* zero_rows, uint32_t* ctrl,
                          int clear_words, float exact_k, hipStream_t s) {
  if (nblk == 0) return hipSuccess;
  dim3 grid(nblk), block(kProjThreads);
  const int cw = clear_words;
  switch (deg) {
    case 0: k_project<0><<<grid, block, 0, s>>>(g, vt, ru, tile, rec, blocksums, nblk, zero_rows, ctrl, cw, exact_k); break;
    case 1: k_project<1><<<grid, block, 0, s>>>(g, vt, ru, tile, rec, blocksums, nblk, zero_rows, ctrl, cw, exact_k); break;
    case 2: k_project<2><<<grid, block, 0, s>>>(g, vt, ru, tile, rec, blocksums, nblk, zero_rows, ctrl, cw, exact_k); break;
    default: k_project<3><<<grid, block, 0, s>>>(g, vt, ru, tile, rec, blocksums, nblk, zero_rows, ctrl, cw, exact_k); break;
  }
  return hipGetLastError();
}

hipError_t launch_scan_small(uint32_t* a, int count, unsigned long long* total, hipStream_t s) {
  k_scan_u32<<<1, 1024, 0, s>>>(a, count, total);
  return hipGetLastError();
}

int64_t scan_pairs_words(int64_t count) {  // (two 64-bit sums, two of a's elements, a tile)
  return count + (count > kSumMany ? 2 * ((count + kSumTile - 1) / kSumTile) : 0);
}

hipError_t launch_scan_pairs(uint2* blocksums, int64_t count, unsigned long long* totals, unsigned long long* host,
                             hipStream_t s) {
  if (count > kSumMany) {
    const int tiles = blocks_for(count, kSumTile);
    auto* part = reinterpret_cast<unsigned long long*>(blocksums + count);
    k_sum_pairs<<<tiles, kSumTile, 0, s>>>(blocksums, count, part);
    k_scan_pairs_down<<<tiles, kSumTile, 0, s>>>(blocksums, count, part, totals, host);
  } else {
    k_scan_pairs<<<1, 1024, 0, s>>>(blocksums, int(count), totals, host);
  }
  return hipGetLastError();
}

bool compact_scans(int64_t count) { return count <= kSumMany; }

hipError_t launch_compact(int64_t n, int views, const Records& rec, const uint2* blocksums, int nblk,
                          unsigned long long* totals, int64_t cap_M, uint32_t* dkeys, uint32_t* dvals,
                          int64_t cap, uint32_t* overflow, bool raw, uint32_t* vstart, hipStream_t s) {
  if (nblk == 0) return hipSuccess;
  if (raw && !compact_scans(int64_t(views) * nblk)) return hipErrorInvalidValue;
  k_compact<<<dim3(nblk, views), kProjThreads, 0, s>>>(n, rec, blocksums, nblk, totals, cap_M, dkeys, dvals, cap,
                                                        overflow, raw ? 1 : 0, vstart);
  return hipGetLastError();
}

template <int ITEMS, bool FOLD>
static void radix_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout, uint32_t* hist,
                       uint32_t* digit_tot, const uint32_t* vstart, int views, const unsigned long long* count,
                       int64_t cap, const uint32_t* overflow, int shift, int nblk, hipStream_t s, Timer* tm) {
  if (tm) tm->begin(K_RADIX_HIST);
  k_radix_hist<ITEMS, FOLD><<<xcd_grid(nblk), kSortThreads, 0, s>>>(kin, vstart, views, count, cap, overflow, shift, hist, nblk);
  if (tm) tm->end(K_RADIX_HIST);
  if (!FOLD) {
    if (tm) tm->begin(K_RADIX_ROWSCAN);
    k_radix_rowscan<<<kSortDigits, 256, 0, s>>>(hist, nblk, digit_tot);
    if (tm) tm->end(K_RADIX_ROWSCAN);
  }
  if (tm) tm->begin(K_RADIX_SCATTER);
  k_radix_scatter<ITEMS, FOLD><<<xcd_grid(nblk), kSortThreads, 0, s>>>(kin, vin, kout, vout, vstart, views, count, cap, overflow,
                                                               shift, hist, digit_tot, nblk);
  if (tm) tm->end(K_RADIX_SCATTER);
}

static int64_t sort_tiles(int64_t cap, int views, int items) { return cap / (items * kSortThreads) + views; }
int64_t radix_hist_words(int64_t cap, int views) { return sort_tiles(cap, views, kSortItemsFew) * kSortDigits; }

hipError_t launch_radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt, uint32_t* vals_alt,
                             uint32_t* hist, uint32_t* digit_tot, const uint32_t* vstart, int views, int64_t per_view,
                             const unsigned long long* count, int64_t cap, const uint32_t* overflow, int key_bits,
                             bool* result_in_alt, int* passes, hipStream_t s, Timer* tm) {
  const int np = (key_bits + kSortBits - 1) / kSortBits;
  *passes = 0;
  *result_in_alt = false;
  if (cap <= 1 || np == 0) return hipSuccess;
  *passes = np;
  const int64_t most = std::min(cap, per_view);  // keys of a view, at most
  if (most <= kSmallMost) {
    if (tm) tm->begin(K_RADIX_SCATTER);
    if (most <= 4 * kSortThreads)
      k_sort_small<4><<<views, kSortThreads, 0, s>>>(keys, vals, vstart, count, cap, overflow, np);
    else
      k_sort_small<16><<<views, kSortThreads, 0, s>>>(keys, vals, vstart, count, cap, overflow, np);
    if (tm) tm->end(K_RADIX_SCATTER);
    return hipGetLastError();
  }
  auto folds = [&](int items) { return (most + items * kSortThreads - 1) / (items * kSortThreads) <= kSortFold; };
  const int items = folds(kSortItemsFew) ? kSortItemsFew : kSortItems;
  const auto pass = items == kSortItemsFew ? radix_pass<kSortItemsFew, true>
                    : folds(kSortItems)    ? radix_pass<kSortItems, true>
                                           : radix_pass<kSortItems, false>;
  const int nblk = int(sort_tiles(cap, views, items));
  uint32_t* kin = keys;
  uint32_t* vin = vals;
  uint32_t* kout = keys_alt;
  uint32_t* vout = vals_alt;
  for (int p = 0; p < np; ++p) {
    pass(kin, vin, kout, vout, hist, digit_tot, vstart, views, count, cap, overflow, kSortBits * p, nblk, s, tm);
    std::swap(kin, kout);
    std::swap(vin, vout);
  }
  *result_in_alt = (np % 2) == 1;
  return hipGetLastError();
}

BinPlan bin_plan(const ViewTable& vt, int64_t cap_vis, int64_t cap_M, int64_t max_tile_counts) {
  // one round of 256 items per block while the count arrays stay within kMaxBinCounts
  // entries; more rounds (fewer, longer chunks and segments) beyond that
  constexpr int64_t PT = kPlaceThreads;
  BinPlan p{};
  p.rows = vt.total_rows;
  const int64_t max_chunks = std::max<int64_t>(1, kMaxBinCounts / std::max(1, p.rows));
  p.rounds1 = int(std::max<int64_t>(1, (cap_vis + PT * max_chunks - 1) / (PT * max_chunks)));
  p.nch1 = int(std::max<int64_t>(1, (cap_vis + PT * p.rounds1 - 1) / (PT * p.rounds1)));
  const int64_t max_segs = std::max<int64_t>(1024, max_tile_counts / std::max(1, vt.max_tiles_x));
  p.rounds2 = int(std::max<int64_t>(1, (cap_M + PT * max_segs - 1) / (PT * max_segs)));
  const int64_t S2 = PT * int64_t(p.rounds2);
  const int64_t segs = (cap_M + S2 - 1) / S2;
  p.cap_M = cap_M;
  p.cap_seg = segs + p.rows;
  p.cap_flat = int64_t(vt.max_tiles_x) * segs + vt.total_tiles;
  return p;
}

// exclusive scan of a[0, min(*count, cap)) (or of a[0, cap) without count); total to *total
static void scan_u32(uint32_t* a, int64_t cap, const unsigned long long* count, uint32_t* part,
                     unsigned long long* total, hipStream_t s) {
  const int nb = int((cap + kScanTile - 1) / kScanTile);
  k_scan_reduce<<<nb, 256, 0, s>>>(a, cap, count, part);
  k_scan_down<<<nb, 256, 0, s>>>(a, cap, count, part, total);
}

hipError_t launch_bin(const ViewTable& vt, int64_t n, const Records& rec, const uint32_t* dvals,
                      const unsigned long long* nvis, int64_t cap_vis, const BinPlan& plan, uint32_t* vals,
                      uint2* ranges, uint32_t* ctrl, float exact_k, int tile, const uint32_t* hint,
                      uint32_t* order, hipStream_t s, Timer* tm) {
  if (vt.total_tiles == 0) return hipSuccess;
  if (cap_vis == 0 || plan.cap_M == 0 || plan.rows == 0) {
    k_fill_u32<<<blocks_for(int64_t(vt.total_tiles) * 2, 256), 256, 0, s>>>(reinterpret_cast<uint32_t*>(ranges), 0u,
                                                                             int64_t(vt.total_tiles) * 2);
    k_tile_order<<<1, 1024, 0, s>>>(ranges, vt.total_tiles, order);
    return hipGetLastError();
  }
  auto B = [&](int k) { if (tm) tm->begin(k); };
  auto E = [&](int k) { if (tm) tm->end(k); };
  uint32_t* overflow = ctrl + kOverflow;
  const size_t lds_rows = size_t(plan.rows) * 4;
  const int64_t n1 = int64_t(plan.rows) * plan.nch1;
  const int g_segs = int(std::min<int64_t>(plan.cap_seg, 8192));
  B(K_BIN_COUNT);
  k_bin_rows_count<<<xcd_grid(plan.nch1), 256, lds_rows, s>>>(vt, n, rec, dvals, nvis, cap_vis, overflow, plan);
  E(K_BIN_COUNT);
  B(K_BIN_SCAN);
  scan_u32(plan.cnt1, n1, nullptr, plan.part, plan.words, s);
  E(K_BIN_SCAN);
  B(K_BIN_SCATTER);
  k_bin_rows_place<<<xcd_grid(plan.nch1), kPlaceThreads, place_lds(std::min(plan.rows, kPlaceBins)), s>>>(
      vt, n, rec, dvals, nvis, cap_vis, overflow, plan);
  E(K_BIN_SCATTER);
  B(K_BIN_COUNT);
  k_bin_tiles_count<<<g_segs, 256, (size_t(vt.max_tiles_x) + 1) * 4, s>>>(vt, plan, rec, exact_k, tile, hint);
  E(K_BIN_COUNT);
  B(K_BIN_SCAN);
  scan_u32(plan.cntF, plan.cap_flat, plan.words + 2, plan.part, plan.words + 3, s);
  E(K_BIN_SCAN);
  B(K_BIN_SCATTER);
  k_bin_tiles_place<<<g_segs, kPlaceThreads, place_lds(std::min(vt.max_tiles_x, kPlaceBins)), s>>>(
      vt, plan, vals, overflow, ranges, hint ? 1 : 0, order);
  E(K_BIN_SCATTER);
  if (!hint) {  // the order not taken by the placement above
    B(K_TILE_ORDER);
    k_tile_order<<<1, 1024, 0, s>>>(ranges, vt.total_tiles, order);
    E(K_TILE_ORDER);
  }
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t count, hipStream_t s) {
  if (count > 0) k_fill_u32<<<blocks_for(count, 256), 256, 0, s>>>(p, value, count);
  return hipGetLastError();
}

hipError_t launch_first_nonfinite(const GaussDev& g, int sh_degree, uint32_t* first, hipStream_t s) {
  k_fill_u32<<<1, 256, 0, s>>>(first, 0xFFFFFFFFu, 1);
  const int K = (sh_degree + 1) * (sh_degree + 1);
  if (g.n > 0) {
    const int64_t total = g.n * (14 + 3 * int64_t(K - 1));
    k_first_nonfinite<<<int(std::min<int64_t>(blocks_for(total, 256), 4096)), 256, 0, s>>>(g, K, first);
  }
  return hipGetLastError();
}

// Persistent grid: blocks resident at once, at most `cap_per_cu` per compute unit.  blend_fwd
// runs fastest at 2 blocks per CU on one 640x480 view, where its heaviest tiles'
// single-wavefront chains bound it and then share a SIMD with fewer others (60, 64, 70 us at 2,
// 3, 4; tiles of 8, 321x239: 42, 47 at 2, 6), and with many tiles per CU at as many as its registers
// allow (eight views 424, 410, 408 us at 4, 5, 6; sixteen 1752x1168 ones 6.63, 6.29, 6.15 ms; one
// of those 365, 348, 354 us).  Tiles of 8 are one wavefront each: 316, 291, 286, 300 us at 4, 6, 12, 18
// on 1280x960 (19k tiles), 1168, 1084, 1031, 1007 over eight views (67k), but 101, 104, 116 at 4,
// 6, 12 on 640x480 (4,800).  blend_bwd: with many items the blocks in flight hide
// each item's fixed latency and the more the better (tiles of 16, sixteen 1752x1168 views:
// 18.5, 14.0, 12.7 ms at 5, 8, 10 per CU; eight uneven views 1204, 967, 930 us), while on one
// 640x480 view 8 and 10 measure the same (128, 130 us).  Tiles of 8 hit the same few rows from
// many blocks: 68, 80, 108 us at 5, 12, 24 per CU on 321x239 (1,230 tiles), 253, 249, 273 at 5,
// 10, 20 on 640x480 (4,800), but 2800, 2809, 2597 over eight views (67k tiles).
template <auto KERN>
static int resident_blocks(int threads, int cap_per_cu) {
  static int per_cu = -1, cus = 1;  // one pair per kernel
  if (per_cu < 0) {
    int p = 0, c = 0, dev = 0;
    (void)hipGetDevice(&dev);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&p, KERN, threads, 0) != hipSuccess || p < 1) p = 1;
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c < 1) c = 1;
    (void)hipGetLastError();
    cus = c;
    per_cu = p;
  }
  return std::min(per_cu, cap_per_cu) * cus;
}

static int device_cus() {
  static int cus = -1;
  if (cus < 0) {
    int c = 0, dev = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || c < 1) c = 1;
    (void)hipGetLastError();
    cus = c;
  }
  return cus;
}
constexpr int kFwdBlocksPerCU = 2;        // up to kFwdManyTilesPerCU tiles per CU
constexpr int kFwdBlocksPerCUMany = 6;    // beyond
constexpr int kFwd8BlocksPerCUMany = 12;  // tiles of 8 beyond 4 kFwdManyTilesPerCU tiles per CU
constexpr int kFwdManyTilesPerCU = 16;
constexpr int kBwdBlocksPerCU = 5;        // tiles of 8 (one wavefront a block)
constexpr int kBwdBlocksPerCUMany = 20;   // beyond 4 kFwdManyTilesPerCU tiles per CU
constexpr int kBwd2BlocksPerCU = 10;      // tiles of 16 and 32
constexpr int kBwdPixelsPerLane = 2;

template <int TS, int BATCH>
static void blend_fwd_t(const ViewTable& vt, const Rules& ru, const Records& rec, const uint2* ranges,
                        const uint32_t* vals, float* T_final, uint32_t* n_contrib, const TileQueue& q,
                        const Ckpt& ck, hipStream_t s) {
  const int many = kFwdManyTilesPerCU * device_cus();
  const int cap = TS == 8 && vt.total_tiles > 4 * many ? kFwd8BlocksPerCUMany
                  : vt.total_tiles > many              ? kFwdBlocksPerCUMany
                                                       : kFwdBlocksPerCU;
  const int grid = std::min(vt.total_tiles, resident_blocks<k_blend_fwd<TS, BATCH>>(TS * TS, cap));
  k_blend_fwd<TS, BATCH><<<grid, TS * TS, 0, s>>>(vt, ru, rec, ranges, vals, T_final, n_contrib, q, ck);
}

hipError_t launch_count_used(const ViewTable& vt, const Rules& ru, const Records& rec, const uint2* ranges,
                             const uint32_t* vals, const uint32_t* n_contrib, int tile, int64_t total_pix,
                             uint32_t* n_used, hipStream_t s) {
  if (total_pix == 0) return hipSuccess;
  k_count_used<<<unsigned((total_pix + 255) / 256), 256, 0, s>>>(vt, ru, rec, ranges, vals, n_contrib, tile, total_pix,
                                                                 n_used);
  return hipGetLastError();
}

// checkpoints every kCkptStride entries over the first 1024 list entries of each tile
int ckpt_stride(int) { return kCkptStride; }
int ckpt_per_tile(int batch) { return std::max(1, 1024 / ckpt_stride(batch)); }

int64_t bwd_items_cap(int total_tiles, int batch) { return int64_t(total_tiles) * (ckpt_per_tile(batch) + 1); }

hipError_t launch_blend_fwd(int tile, int batch, const ViewTable& vt, const Rules& ru, const Records& rec,
                            const uint2* ranges, const uint32_t* vals, float* T_final, uint32_t* n_contrib,
                            const TileQueue& q, const Ckpt& ck, hipStream_t s) {
  if (vt.total_tiles == 0) return hipSuccess;
  const bool b256 = batch == 256;
  switch (tile) {
    case 8: b256 ? blend_fwd_t<8, 256>(vt, ru, rec, ranges, vals, T_final, n_contrib, q, ck, s)
                 : blend_fwd_t<8, 128>(vt, ru, rec, ranges, vals, T_final, n_contrib, q, ck, s); break;
    case 32: b256 ? blend_fwd_t<32, 256>(vt, ru, rec, ranges, vals, T_final, n_contrib, q, ck, s)
                  : blend_fwd_t<32, 128>(vt, ru, rec, ranges, vals, T_final, n_contrib, q, ck, s); break;
    default: b256 ? blend_fwd_t<16, 256>(vt, ru, rec, ranges, vals, T_final, n_contrib, q, ck, s)
                  : blend_fwd_t<16, 128>(vt, ru, rec, ranges, vals, T_final, n_contrib, q, ck, s); break;
  }
  return hipGetLastError();
}

int loss_partials(const ViewTable& vt) {
  int64_t maxp = 0;
  for (int v = 0; v < vt.nviews; ++v) maxp = std::max<int64_t>(maxp, int64_t(vt.v[v].W) * vt.v[v].H);
  return int(blocks_for(maxp, 256)) * vt.nviews;
}

// the sums of the queue's slices, where list_bwd_items reads them
static void launch_items_sum(const ViewTable& vt, int stride, const uint32_t* order, const Ckpt& ck, hipStream_t s) {
  if (vt.total_tiles > kListExact)
    k_items_sum<<<blocks_for(vt.total_tiles, 256), 256, 0, s>>>(order, vt.total_tiles, stride, ck);
}

hipError_t launch_loss_l1(const ViewTable& vt, float depth_w, float* part, float* loss, hipStream_t s,
                          const uint32_t* order, int batch, const Ckpt* ck, uint32_t* ctrl, uint32_t* host_flag) {
  const int np = loss_partials(vt);
  if (order) launch_items_sum(vt, ckpt_stride(batch), order, *ck, s);
  k_loss_l1<<<dim3(np / vt.nviews, vt.nviews), 256, 0, s>>>(vt, depth_w, part, order, vt.total_tiles,
                                                            ckpt_stride(batch), ck ? *ck : Ckpt{}, ctrl, host_flag);
  if (loss) k_loss_sum<<<1, 256, 0, s>>>(part, np, loss);
  return hipGetLastError();
}

template <int TS>
static void blend_bwd_t(const ViewTable& vt, const Rules& ru, const Records& rec, const uint2* ranges,
                        const uint32_t* vals, const float* T_final, const uint32_t* n_contrib, float* grad2d,
                        const TileQueue& q, const Ckpt& ck, hipStream_t s) {
  constexpr int PPL = TS >= 16 ? kBwdPixelsPerLane : 1;
  const int cap = TS >= 16 ? kBwd2BlocksPerCU
                  : vt.total_tiles > 4 * kFwdManyTilesPerCU * device_cus() ? kBwdBlocksPerCUMany : kBwdBlocksPerCU;
  const int grid =
      int(std::min<int64_t>(ck.cap_items, resident_blocks<k_blend_bwd2<TS, PPL>>(TS * TS / PPL, cap)));
  k_blend_bwd2<TS, PPL><<<grid, TS * TS / PPL, 0, s>>>(vt, ru, rec, ranges, vals, T_final, n_contrib, grad2d, q, ck);
}

hipError_t launch_blend_bwd(int tile, int batch, const ViewTable& vt, const Rules& ru, const Records& rec,
                            const uint2* ranges, const uint32_t* vals, const float* T_final,
                            const uint32_t* n_contrib, float* grad2d, const TileQueue& q, const Ckpt& ck,
                            hipStream_t s, bool items_listed) {
  if (vt.total_tiles == 0) return hipSuccess;
  if (!items_listed) {
    launch_items_sum(vt, ckpt_stride(batch), q.order, ck, s);
    k_bwd_items<<<blocks_for(vt.total_tiles, 256), 256, 0, s>>>(q.order, vt.total_tiles, ckpt_stride(batch), ck, q.ctrl);
  }
  switch (tile) {
    case 8: blend_bwd_t<8>(vt, ru, rec, ranges, vals, T_final, n_contrib, grad2d, q, ck, s); break;
    case 32: blend_bwd_t<32>(vt, ru, rec, ranges, vals, T_final, n_contrib, grad2d, q, ck, s); break;
    default: blend_bwd_t<16>(vt, ru, rec, ranges, vals, T_final, n_contrib, grad2d, q, ck, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_project_bwd(int deg, const GaussDev& g, const ViewTable& vt, const Rules& ru,
                              const Records& rec, const float* grad2d, float* dp_sh, const GradOut& out,
                              const AdamDev& adam, hipStream_t s, const float* loss_part, int loss_np,
                              float* loss) {
  if (g.n == 0) return hipSuccess;
  const dim3 gsh(blocks_for(g.n, kShGaussians));
  switch (deg) {
    case 0: k_project_bwd_sh<0><<<gsh, 256, 0, s>>>(g, vt, rec, grad2d, out, dp_sh, adam); break;
    case 1: k_project_bwd_sh<1><<<gsh, 256, 0, s>>>(g, vt, rec, grad2d, out, dp_sh, adam); break;
    case 2: k_project_bwd_sh<2><<<gsh, 256, 0, s>>>(g, vt, rec, grad2d, out, dp_sh, adam); break;
    default: k_project_bwd_sh<3><<<gsh, 256, 0, s>>>(g, vt, rec, grad2d, out, dp_sh, adam); break;
  }
  k_project_bwd_geo<<<blocks_for(g.n, kProjThreads), kProjThreads, 0, s>>>(g, vt, ru, rec, grad2d, dp_sh, out,
                                                                           adam, loss_part, loss_np, loss);
  return hipGetLastError();
}

}  // namespace gsr
