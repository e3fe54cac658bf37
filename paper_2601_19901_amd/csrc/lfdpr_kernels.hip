// HIP kernels of the LFDPR hot path for gfx950 (wave64).
//
//   k_tri_setup   one lane per triangle (eight in small scenes): frame transform, visibility in every
//                 LFD view, T_align frame, LFD-biased H/V densities, Eqs. 1-7,
//                 lattice snap, cell count (rows over the workgroup's
//                 lanes); each workgroup's count sum and the list of
//                 triangles with many cells                    (Sec. 3, 3.1, 3.3)
//   k_scan_top    one workgroup: the workgroups' count sums -> point offset bases
//   k_emit        point offsets, and the cells in deterministic order, one
//                 lane per lattice row; triangles with many cells: one
//                 workgroup each (same launch)
//   k_fetch       one lane per point: UV at the cell centre, two trilinear
//                 mip fetches (tv_min, tv_max)                (Sec. 3.3); for
//                 the triangle-view order and the quilt also the point's
//                 splat rectangle (and, for the quilt, its pixel rows)
//   k_splat       a wave takes 64 points through the views: splat boxes, then
//                 their covered pixels 64 at a time: cell ownership, Eqs. 8-9,
//                 64-bit atomicMin of (depth, colour)         (Sec. 3.2, 3.3, 5.1)
//   k_qcount, k_qplan, k_qscatter   the quilt's band lists: points binned by
//                 the pixel rows their splat reaches           (Sec. 3.2)
//   k_splat_quilt one workgroup per tile (a band of rows x a subset of the
//                 views): the same splat with the 64-bit keys in LDS, the
//                 tile written out as RGBA8 (+ depth)          (Sec. 3.2, 5.1)
//   k_splat_tv    per (triangle, view): covered pixels find their owning point
//   k_resolve     keys -> RGBA8 (+ depth), keys re-cleared for the next frame
//   k_interleave  one lane per four panel pixels: tilted-lens phase, view and
//                 pixel index, optional 8-tap Gaussian reconstruction (Sec. 4)
//   k_angular_filter  sub-views -> views (angular supersampling, Sec. 4), one
//                 lane per four pixels
#include "lfdpr_device.h"
#include "lfdpr_internal.h"

namespace lfdpr {

// ------------------------------------------------------------------ utilities

// wave64 inclusive scan of one uint64 per lane
__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    uint64_t o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

__device__ __forceinline__ uint64_t wave_sum(uint64_t v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

__global__ void k_fill_u64(uint64_t* __restrict__ p, int64_t n, uint64_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// The single-frame item table, written from a kernel argument (no host staging).
__global__ void k_store_item(Item it, Item* __restrict__ dst) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = it;
}

// Frame statistics for the caller: points, active triangles, point-views,
// overflowed triangles, written pixels, point capacity.
__global__ void __launch_bounds__(64) k_export_stats(const uint64_t* __restrict__ st, int64_t cap,
                                                      int64_t* __restrict__ out) {
  static_assert(kWorkQueues == 64, "a line per lane");
  const uint64_t written = wave_sum(st[kStatLines + LINE_WORDS * threadIdx.x + LINE_WRITTEN]);
  if (threadIdx.x == 0) {
    out[0] = (int64_t)st[STAT_TOTAL];
    out[1] = (int64_t)st[STAT_ACTIVE];
    out[2] = (int64_t)st[STAT_POINT_VIEWS];
    out[3] = (int64_t)st[STAT_OVERFLOW];
    out[4] = (int64_t)written;
    out[5] = cap;
  }
}

__global__ void k_build_mip(const uint32_t* __restrict__ src, uint32_t* __restrict__ dst, int s) {
  int h = s >> 1;
  int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= (int64_t)h * h) return;
  int y = (int)(k / h), x = (int)(k % h);
  uint32_t a = src[(int64_t)(2 * y) * s + 2 * x], b = src[(int64_t)(2 * y) * s + 2 * x + 1];
  uint32_t c = src[(int64_t)(2 * y + 1) * s + 2 * x], d = src[(int64_t)(2 * y + 1) * s + 2 * x + 1];
  uint32_t r = 0;
#pragma unroll
  for (int ch = 0; ch < 4; ++ch) {
    int sh = 8 * ch;
    uint32_t m = (((a >> sh) & 255u) + ((b >> sh) & 255u) + ((c >> sh) & 255u) + ((d >> sh) & 255u) + 2u) >> 2;
    r |= m << sh;
  }
  dst[k] = r;
}

// Adds a wave's `v` to the wave's line of a statistic (one lane calls).
__device__ __forceinline__ void line_add(uint64_t* stats, int slot, uint64_t v) {
  const uint32_t line = (blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) % kWorkQueues;
  if (v) atomicAdd((unsigned long long*)(stats + kStatLines + LINE_WORDS * line + slot), (unsigned long long)v);
}

// Slot of this lane in a list shared by the grid when `take`: one atomic per wave.
__device__ __forceinline__ uint64_t wave_append(bool take, uint64_t* counter) {
  const uint64_t mask = __builtin_amdgcn_ballot_w64(take);
  if (!mask) return 0;
  const int lane = threadIdx.x & 63;
  const int leader = __builtin_ctzll(mask);
  uint64_t base = 0;
  if (lane == leader) base = atomicAdd((unsigned long long*)counter, (unsigned long long)__builtin_popcountll(mask));
  base = __shfl(base, leader, 64);
  const uint64_t below = lane ? (mask & (~0ull >> (64 - lane))) : 0ull;
  return base + (uint64_t)__builtin_popcountll(below);
}

// Exclusive prefix of v over the 256 lanes of the workgroup (every lane calls).
__device__ __forceinline__ uint64_t block_excl_scan(uint64_t v, uint64_t* ws4) {
  const uint64_t inc = wave_incl_scan(v);
  if ((threadIdx.x & 63) == 63) ws4[threadIdx.x >> 6] = inc;
  __syncthreads();
  uint64_t before = 0;
  for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) before += ws4[w];
  __syncthreads();  // ws4 may be rewritten after this
  return before + inc - v;
}

// Sum of v over the 256 lanes of the workgroup (every lane calls).
__device__ __forceinline__ uint64_t block_sum(uint64_t v, uint64_t* ws4) {
  const uint64_t w = wave_sum(v);
  if ((threadIdx.x & 63) == 0) ws4[threadIdx.x >> 6] = w;
  __syncthreads();
  const uint64_t sum = (ws4[0] + ws4[1]) + (ws4[2] + ws4[3]);
  __syncthreads();  // ws4 may be rewritten after this
  return sum;
}

// ------------------------------------------------------------------ a1/a2: triangle setup

// Smallest value and sum over a group of kVL neighbouring lanes.
template <int kVL>
__device__ __forceinline__ float group_min(float v) {
#pragma unroll
  for (int d = kVL / 2; d >= 1; d >>= 1) v = fminf(v, __shfl_xor(v, d, 64));
  return v;
}
template <int kVL>
__device__ __forceinline__ int group_sum(int v) {
#pragma unroll
  for (int d = kVL / 2; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// Visibility and LFD-biased densities (Sec. 3.1) over views first, first +
// step, .. of the rig: the number of active views, the smallest pixel edges and
// footprint, and the smallest and (negated) largest plane distance.
struct ViewSums {
  int nact;
  float lx, ly, A, ad_lo, ad_hi_neg;
};
template <bool kPlain>
__device__ __forceinline__ ViewSums sum_views(const Rig& rg, const TriRec& R, F3 P0, F3 P1, F3 P2, int first, int step,
                                              uint32_t* odd) {
  ViewSums S{0, INFINITY, INFINITY, INFINITY, INFINITY, 0.0f};
  const float p0y2 = P0.y * P0.y, p0z2 = P0.z * P0.z;
  // x * 256 < -0.5 rounds below 0; x * 256 > 256 W + 0.5 rounds above 256 W
  const float x_left = -0.5f / 256.0f, x_right = ((float)(256 * rg.W) + 0.5f) / 256.0f;
  const Divisor dfx = divisor(rg.fx), dfy = divisor(rg.fy);
  // the next view's eye offset is fetched one iteration ahead
  float b_next = first < rg.n_views ? rg.eye[first] : 0.0f;
  for (int r = first; r < rg.n_views; r += step) {
    const float b = b_next;
    if (r + step < rg.n_views) b_next = rg.eye[r + step];
    // view_active(), whose conditions on the projected rows are settled by may_be_seen()
    const float delta = R.h - R.nx * b;
    if (!faces_eye(P0.x, p0y2, p0z2, delta, b)) continue;
    const float x0 = R.a0 - b * R.c0, x1 = R.a1 - b * R.c1, x2 = R.a2 - b * R.c2;
    if (!(fabsf(x0) < kGuard) || !(fabsf(x1) < kGuard) || !(fabsf(x2) < kGuard)) continue;
    if (fmaxf(x0, fmaxf(x1, x2)) < x_left || fminf(x0, fminf(x1, x2)) > x_right) continue;
    ++S.nact;
    const F3 e{b, 0.0f, 0.0f};
    const F3 Ps = nearest_on_triangle<kPlain>(e, P0, P1, P2, odd);
    const F3 d = sub3(Ps, e);
    const float ad = fabsf(delta), Zs = Ps.z;
    const Divisor dd = divisor(delta);
    const float g = kPlain ? quotient(R.nx, dd) : R.nx / delta;
    const float vx = 1.0f - d.x * g, vy = 0.0f - d.y * g, vz = 0.0f - d.z * g;
    const float vv = (vx * vx + vy * vy) + vz * vz;
    const float lx = (kPlain ? quotient(Zs, dfx) : Zs / rg.fx) * (kPlain ? root(vv) : sqrtf(vv));
    const float g2 = kPlain ? quotient(R.ny, dd) : R.ny / delta;
    const float wx = 0.0f - d.x * g2, wy = 1.0f - d.y * g2, wz = 0.0f - d.z * g2;
    const float ww = (wx * wx + wy * wy) + wz * wz;
    const float ly = (kPlain ? quotient(Zs, dfy) : Zs / rg.fy) * (kPlain ? root(ww) : sqrtf(ww));
    const float fa = rg.fxfy * ad, z3 = (Zs * Zs) * Zs;
    const float A = kPlain ? quotient(z3, divisor(fa)) : z3 / fa;
    S.lx = lx < S.lx ? lx : S.lx;
    S.ly = ly < S.ly ? ly : S.ly;
    S.A = A < S.A ? A : S.A;
    S.ad_lo = ad < S.ad_lo ? ad : S.ad_lo;
    S.ad_hi_neg = -ad < S.ad_hi_neg ? -ad : S.ad_hi_neg;
  }
  return S;
}

// kMulti: triangles of several items (a batch), each lane finds its own; else
// every triangle belongs to items[0], whose rig then sits in scalar registers.
// kVL lanes share a triangle and split its views (setup_lanes).
//
// The view loop (sum_views) issues most of the instructions: six quotients and
// two roots per active view, by quotient() and root() where the operands allow.
// The records are stored before the cells are counted and the rows of the
// workgroup's lattices are spread over its lanes: a lane that counts its own
// triangle's rows holds its wave for the largest of 64, with the whole record
// in registers meanwhile (158 instead of 86).  Measured, before -> now: 1.0M
// triangles and 192 views 657 -> 478 us, 0.18M and 25 views 99 -> 81, 1,280
// triangles and 8 views 26.5 -> 14.4 us (eight lanes each).
template <bool kMulti, int kVL>
__global__ void __launch_bounds__(256) k_tri_setup(SetupArgs a) {
  constexpr int kTris = 256 / kVL;
  __shared__ int4 l_st[kTris];        // s1, t1, s2, t2
  __shared__ int32_t l_j0[kTris];     // first row of the lattice's box
  __shared__ uint32_t l_rows[kTris];  // its rows, then the rows before this triangle's
  __shared__ uint32_t l_cnt[kTris];
  __shared__ int32_t l_jlo[kTris], l_jhi[kTris];
  __shared__ uint32_t l_odd[256];     // a lane's view loop met a nearest point off its triangle
  __shared__ uint64_t ws4[4];
  const int tl = threadIdx.x / kVL, sub = threadIdx.x % kVL;
  const int64_t t = (int64_t)blockIdx.x * kTris + tl;
  uint64_t act_cnt = 0, ovf_cnt = 0, pv_cnt = 0;
  uint32_t cnt = 0;
  int nact = 0;
  bool ovf = false;
  int32_t nrows = 0;
  if (t < a.nt) {
    if (a.dbgf && sub == 0) {
      for (int k = 0; k < 8; ++k) { a.dbgf[t * 8 + k] = 0.0f; a.dbgi[t * 8 + k] = 0; }
    }
    const int item = kMulti ? find_item(a.items, a.n_items, t) : 0;
    const Item& it = a.items[item];
    const int64_t lt = t - it.tri_base;
    const Rig rg = it.rig;  // in registers: the view loop reads it every iteration
    const float* m = a.models ? a.models[item].m : a.model.m;
    float P[3][3];
    bool ok = true;
    uint32_t vi[3];
    for (int k = 0; k < 3; ++k) {
      vi[k] = it.idx[lt * 3 + k];
      float px = it.pos[(int64_t)vi[k] * 3], py = it.pos[(int64_t)vi[k] * 3 + 1], pz = it.pos[(int64_t)vi[k] * 3 + 2];
      P[k][0] = ((m[0] * px + m[1] * py) + m[2] * pz) + m[3];
      P[k][1] = ((m[4] * px + m[5] * py) + m[6] * pz) + m[7];
      P[k][2] = ((m[8] * px + m[9] * py) + m[10] * pz) + m[11];
      if (!(P[k][2] >= rg.znear)) ok = false;
    }
    F3 P0{P[0][0], P[0][1], P[0][2]}, P1{P[1][0], P[1][1], P[1][2]}, P2{P[2][0], P[2][1], P[2][2]};
    F3 e1 = sub3(P1, P0), e2 = sub3(P2, P0);
    F3 n{e1.y * e2.z - e1.z * e2.y, e1.z * e2.x - e1.x * e2.z, e1.x * e2.y - e1.y * e2.x};
    float nl = sqrtf((n.x * n.x + n.y * n.y) + n.z * n.z);
    if (ok && (!(nl > 0.0f) || isinf(nl))) ok = false;
    TriRec R;
    if (ok) {
      R.nx = n.x / nl; R.ny = n.y / nl; R.nz = n.z / nl;
      R.p0x = P0.x; R.p0y = P0.y; R.p0z = P0.z;
      R.h = (R.nx * P0.x + R.ny * P0.y) + R.nz * P0.z;
      vertex_proj(rg, P0.x, P0.y, P0.z, R.a0, R.c0, R.y0);
      vertex_proj(rg, P1.x, P1.y, P1.z, R.a1, R.c1, R.y1);
      vertex_proj(rg, P2.x, P2.y, P2.z, R.a2, R.c2, R.y2);
    }
    // triangles that no view can see skip the view loop (see may_be_seen)
    const bool seen = ok && may_be_seen(rg, R);
    // the wave's view loops in the middle of the binary32 range, or with the plain operators
    float far = fmaxf(fabsf(rg.eye_lo), fabsf(rg.eye_hi));
    for (int k = 0; k < 3; ++k)
      for (int q = 0; q < 3; ++q) far = fmaxf(far, fabsf(P[k][q]));
    const float zlo = fminf(P[0][2], fminf(P[1][2], P[2][2]));
    const bool plain = __builtin_amdgcn_ballot_w64(seen && !plain_operands(rg, zlo, far)) == 0;
    ViewSums S{0, INFINITY, INFINITY, INFINITY, INFINITY, 0.0f};
    uint32_t* const odd = &l_odd[threadIdx.x];  // in LDS: the loop has no register for it to merge at each view
    *odd = 0u;
    if (plain && seen) S = sum_views<true>(rg, R, P0, P1, P2, sub, kVL, odd);
    if (!plain || __builtin_amdgcn_ballot_w64(*odd != 0u)) {
      if (seen) S = sum_views<false>(rg, R, P0, P1, P2, sub, kVL, odd);
    }
    nact = group_sum<kVL>(S.nact);
    const float lxmin = group_min<kVL>(S.lx), lymin = group_min<kVL>(S.ly), Amin = group_min<kVL>(S.A);
    const float admin = group_min<kVL>(S.ad_lo), admax = 0.0f - group_min<kVL>(S.ad_hi_neg);
    if (ok && nact > 0) {
      act_cnt = sub == 0 ? 1 : 0;
      // T_align: s axis = camera X projected into the plane, t axis = n x s
      float upx, upy, upz;
      if (fabsf(R.nx) > 0.99999f) {
        upx = 0.0f - R.nx * R.ny; upy = 1.0f - R.ny * R.ny; upz = 0.0f - R.nz * R.ny;
      } else {
        upx = 1.0f - R.nx * R.nx; upy = 0.0f - R.ny * R.nx; upz = 0.0f - R.nz * R.nx;
      }
      float ul = sqrtf((upx * upx + upy * upy) + upz * upz);
      R.ux = upx / ul; R.uy = upy / ul; R.uz = upz / ul;
      R.wx = R.ny * R.uz - R.nz * R.uy;
      R.wy = R.nz * R.ux - R.nx * R.uz;
      R.wz = R.nx * R.uy - R.ny * R.ux;
      float Sx = 1.0f / lxmin, Sy = 1.0f / lymin;
      float size_xy = Amin;
      // texture-based sampling, Eqs. 1-3
      const int tex = it.tex[lt];
      const TexInfo& ti = it.texinfo[tex];
      // physically based mode: three more textures; Eq. 1 takes the largest
      const bool pbr = a.tm != nullptr;
      int32_t texk[4] = {tex, tex, tex, tex};
      if (pbr) {
        texk[1] = it.mat[lt * 3];
        texk[2] = it.mat[lt * 3 + 1];
        texk[3] = it.mat[lt * 3 + 2];
      }
      float uv0u = it.uv[(int64_t)vi[0] * 2], uv0v = it.uv[(int64_t)vi[0] * 2 + 1];
      float du1 = it.uv[(int64_t)vi[1] * 2] - uv0u, dv1 = it.uv[(int64_t)vi[1] * 2 + 1] - uv0v;
      float du2 = it.uv[(int64_t)vi[2] * 2] - uv0u, dv2 = it.uv[(int64_t)vi[2] * 2 + 1] - uv0v;
      float Ats = 0.5f * fabsf(du1 * dv2 - dv1 * du2);
      float Aws = 0.5f * nl;
      float Xt = (float)ti.size;
      float ntex = (Ats * Xt) * Xt;
      if (pbr) {
        for (int k = 1; k < 4; ++k) {
          const float Xk = (float)it.texinfo[texk[k]].size;
          const float nk = (Ats * Xk) * Xk;
          ntex = nk > ntex ? nk : ntex;
        }
      }
      if (ntex > 0.0f) {
        float size_uv = Aws / ntex;
        if (size_uv > size_xy) {
          float f = sqrtf(size_xy / size_uv);
          Sx = Sx * f;
          Sy = Sy * f;
        }
      }
      R.sx = Sx; R.sy = Sy;
      R.ruv = Ats / Aws;
      // multiview-mip setup, Eqs. 4-7
      float Zmin = P0.z, Zmax = P0.z;
      Zmin = P1.z < Zmin ? P1.z : Zmin; Zmax = P1.z > Zmax ? P1.z : Zmax;
      Zmin = P2.z < Zmin ? P2.z : Zmin; Zmax = P2.z > Zmax ? P2.z : Zmax;
      R.smin = (((Zmin * Zmin) * Zmin) / (rg.fxfy * admax)) * R.ruv;
      R.smax = (((Zmax * Zmax) * Zmax) / (rg.fxfy * admin)) * R.ruv;
      R.irange = R.smax > R.smin ? 1.0f / (R.smax - R.smin) : 0.0f;
      R.cu0 = R.uy * P0.y + R.uz * P0.z;
      R.cw0 = R.wy * P0.y + R.wz * P0.z;
      R.item = item;
      R.pad1 = 0;
      int32_t kmin = 0, kmax = 0;
      if (rg.mip) {
        int32_t top = 256 * (ti.levels - 1);
        kmin = lod_q8(a.lod_thr, (R.smin * Xt) * Xt);
        kmax = lod_q8(a.lod_thr, (R.smax * Xt) * Xt);
        kmin = kmin < 0 ? 0 : (kmin > top ? top : kmin);
        kmax = kmax < 0 ? 0 : (kmax > top ? top : kmax);
      }
      TriMat M{};
      if (pbr) {
        // Eqs. 6-7 for each material texture at its own size and level count
        int32_t kq[6] = {0, 0, 0, 0, 0, 0};
        if (rg.mip) {
          for (int k = 1; k < 4; ++k) {
            const TexInfo& tk = it.texinfo[texk[k]];
            const float Xk = (float)tk.size;
            const int32_t top = 256 * (tk.levels - 1);
            int32_t k0 = lod_q8(a.lod_thr, (R.smin * Xk) * Xk);
            int32_t k1 = lod_q8(a.lod_thr, (R.smax * Xk) * Xk);
            kq[2 * k - 2] = k0 < 0 ? 0 : (k0 > top ? top : k0);
            kq[2 * k - 1] = k1 < 0 ? 0 : (k1 > top ? top : k1);
          }
        }
        F3 Tf, Bf;
        texture_frame(e1, e2, du1, dv1, du2, dv2, F3{R.nx, R.ny, R.nz}, F3{R.ux, R.uy, R.uz},
                      F3{R.wx, R.wy, R.wz}, Tf, Bf);
        M.texn = texk[1]; M.texr = texk[2]; M.texm = texk[3];
        M.kn0 = kq[0]; M.kn1 = kq[1]; M.kr0 = kq[2]; M.kr1 = kq[3]; M.km0 = kq[4]; M.km1 = kq[5];
        M.tx = Tf.x; M.ty = Tf.y; M.tz = Tf.z; M.bx = Bf.x; M.by = Bf.y; M.bz = Bf.z;
      }
      // sample lattice, vertex 0 at the centre of cell (0,0)
      int32_t sq[3] = {128, 0, 0}, tq[3] = {128, 0, 0};
      F3 ek[2] = {e1, e2};
      F3 uh{R.ux, R.uy, R.uz}, wh{R.wx, R.wy, R.wz};
      for (int k = 0; k < 2; ++k) {
        float s = Sx * dot3(uh, ek[k]) + 0.5f;
        float tt = Sy * dot3(wh, ek[k]) + 0.5f;
        if (!(fabsf(s) < 16384.0f) || !(fabsf(tt) < 16384.0f)) { ovf = true; break; }
        sq[k + 1] = (int32_t)rintf(s * 256.0f);
        tq[k + 1] = (int32_t)rintf(tt * 256.0f);
      }
      if (a.dbgf && sub == 0) {
        float* df = a.dbgf + t * 8;
        int32_t* di = a.dbgi + t * 8;
        df[0] = Sx; df[1] = Sy; df[2] = R.smin; df[3] = R.smax; df[4] = R.ruv; df[5] = R.h;
        df[6] = size_xy; df[7] = (float)nact;
        if (!ovf) { di[0] = sq[1]; di[1] = tq[1]; di[2] = sq[2]; di[3] = tq[2]; }
        di[4] = kmin; di[5] = kmax; di[6] = 1;
      }
      if (!ovf) {
        Lattice L;
        lattice_init(L, sq[1], tq[1], sq[2], tq[2]);
        if ((L.iB - L.iA + 1) * (L.jB - L.jA + 1) > kBoxCap) ovf = true;
        else nrows = (int32_t)(L.jB - L.jA + 1);
        if (sub == 0 && nrows) {
          TriEmit E;
          E.uv0u = uv0u; E.uv0v = uv0v; E.du1 = du1; E.dv1 = dv1; E.du2 = du2; E.dv2 = dv2;
          E.s1 = sq[1]; E.t1 = tq[1]; E.s2 = sq[2]; E.t2 = tq[2];
          E.kmin = kmin; E.kmax = kmax; E.tex = tex; E.item = item;
          E.jlo = 0; E.jhi = -1;
          a.rec[t] = R;
          a.em[t] = E;
          if (pbr) a.tm[t] = M;
          l_st[tl] = make_int4(sq[1], tq[1], sq[2], tq[2]);
          l_j0[tl] = (int32_t)L.jA;
        }
      }
    }
  }
  // the rows of the workgroup's lattices, spread over its lanes
  if (sub == 0) {
    l_cnt[tl] = 0u;
    l_jlo[tl] = 0x7FFFFFFF;
    l_jhi[tl] = -0x7FFFFFFF;
  }
  const uint32_t before = (uint32_t)block_excl_scan(sub == 0 ? (uint64_t)nrows : 0ull, ws4);
  if (sub == 0) l_rows[tl] = before;
  const uint32_t total = (uint32_t)block_sum(sub == 0 ? (uint64_t)nrows : 0ull, ws4);
  for (uint32_t k = threadIdx.x; k < total; k += 256) {
    int q = 0;  // the last triangle whose rows begin at or before k: it has some
#pragma unroll
    for (int st = kTris / 2; st >= 1; st >>= 1)
      if (l_rows[q + st] <= k) q += st;
    const int4 st = l_st[q];
    Lattice L;
    lattice_init(L, st.x, st.y, st.z, st.w);
    const int64_t j = (int64_t)l_j0[q] + (int64_t)(k - l_rows[q]);
    int64_t lo, hi;
    lattice_row(L, j, lo, hi);
    if (hi >= lo) {
      atomicAdd(&l_cnt[q], (uint32_t)(hi - lo + 1));
      atomicMin(&l_jlo[q], (int32_t)j);
      atomicMax(&l_jhi[q], (int32_t)j);
    }
  }
  __syncthreads();
  if (t < a.nt && sub == 0) {
    if (nrows) {
      cnt = l_cnt[tl];
      if (cnt > (uint32_t)kCellCap) ovf = true;
    }
    if (ovf) {
      cnt = 0;
      ovf_cnt = 1;
      if (a.dbgi) a.dbgi[t * 8 + 7] = 1;
    }
    pv_cnt = (uint64_t)cnt * (uint64_t)nact;
    if (cnt > 0) *reinterpret_cast<int2*>(&a.em[t].jlo) = make_int2(l_jlo[tl], l_jhi[tl]);
    a.counts[t] = cnt;
  }
  // triangles with more cells than one lane emits go to the workgroup list
  const bool big = cnt > kBigCells;
  const uint64_t bslot = wave_append(big, a.n_big);
  if (big) a.big[bslot] = (uint32_t)t;
  // this workgroup's points and statistics; k_scan_top adds them up (three
  // counters of the whole launch took longer than the set-up itself: 16 thousand
  // waves at 1.0M triangles, 301 -> 171 us)
  const uint64_t points = block_sum((uint64_t)cnt, ws4);
  const uint64_t stat = block_sum(pv_cnt | (act_cnt << 36) | (ovf_cnt << 50), ws4);
  if (threadIdx.x == 0) {
    a.tile_sum[blockIdx.x] = points;
    a.tile_stat[blockIdx.x] = stat;
  }
  if (kVL == 8 && a.ticket) {  // the last workgroup to get here does the work of k_scan_top
    __shared__ bool last;
    if (threadIdx.x == 0)
      last = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (!last) return;
    uint64_t sum = 0, q = 0;
    if (threadIdx.x < gridDim.x) {
      sum = __hip_atomic_load(a.tile_sum + threadIdx.x, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
      q = __hip_atomic_load(a.tile_stat + threadIdx.x, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint64_t base = block_excl_scan(sum, ws4);
    if (threadIdx.x < gridDim.x) a.tile_sum[threadIdx.x] = base;
    const uint64_t all = block_sum(sum, ws4), pv = block_sum(q & ((1ull << 36) - 1), ws4);
    const uint64_t act = block_sum((q >> 36) & 0x3FFFu, ws4), over = block_sum(q >> 50, ws4);
    if (threadIdx.x == 0) {
      a.stats[STAT_TOTAL] = all;
      a.stats[STAT_POINT_VIEWS] = pv;
      a.stats[STAT_ACTIVE] = act;
      a.stats[STAT_OVERFLOW] = over;
    }
  }
}

// ------------------------------------------------------------------ scan (counts -> offsets)
// The point offsets are an exclusive prefix sum of the per-triangle counts: each
// set-up workgroup writes the sum of its triangles, k_scan_top turns the sums
// into bases (one workgroup; also the grand total), and the emission kernel
// adds the prefix within its tile, the triangles of one set-up workgroup.  Up to kScanTiles set-up workgroups, one sum per thread, the last
// of them to finish does it instead of a launch (a frame of 1,280 triangles 53.1
// -> 51.4 us).
__global__ void __launch_bounds__(1024) k_scan_top(uint64_t* __restrict__ tile_sum,
                                                    const uint64_t* __restrict__ tile_stat, int64_t ntiles,
                                                    uint64_t* __restrict__ stats) {
  __shared__ uint64_t ws[16], st[16][3];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  // a run of tiles per thread: its sum, a scan over the threads, its bases
  const int64_t per = (ntiles + 1023) / 1024, t0 = imin(ntiles, per * threadIdx.x), t1 = imin(ntiles, t0 + per);
  uint64_t sum = 0, pv = 0, act = 0, ovf = 0;
#pragma unroll 4
  for (int64_t t = t0; t < t1; ++t) {
    sum += tile_sum[t];
    const uint64_t q = tile_stat[t];
    pv += q & ((1ull << 36) - 1);
    act += (q >> 36) & 0x3FFFu;
    ovf += q >> 50;
  }
  const uint64_t inc = wave_incl_scan(sum);
  pv = wave_sum(pv);
  act = wave_sum(act);
  ovf = wave_sum(ovf);
  if (lane == 63) ws[wv] = inc;
  if (lane == 0) {
    st[wv][0] = pv;
    st[wv][1] = act;
    st[wv][2] = ovf;
  }
  __syncthreads();
  uint64_t run = inc - sum, total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wv) run += ws[w];
    total += ws[w];
  }
#pragma unroll 4
  for (int64_t t = t0; t < t1; ++t) {
    const uint64_t v = tile_sum[t];
    tile_sum[t] = run;
    run += v;
  }
  if (threadIdx.x == 0) {
    stats[STAT_TOTAL] = total;
    pv = act = ovf = 0;
    for (int w = 0; w < 16; ++w) {
      pv += st[w][0];
      act += st[w][1];
      ovf += st[w][2];
    }
    stats[STAT_POINT_VIEWS] = pv;
    stats[STAT_ACTIVE] = act;
    stats[STAT_OVERFLOW] = ovf;
  }
}

// ------------------------------------------------------------------ a1/a2: emission

__device__ __forceinline__ void write_head(Point* pts, uint64_t gi, uint32_t t, uint32_t f, int64_t i, int64_t j) {
  uint2 head;
  head.x = t | (f << 28);
  head.y = (uint32_t)(uint16_t)(int16_t)i | ((uint32_t)(uint16_t)(int16_t)j << 16);
  *reinterpret_cast<uint2*>(&pts[gi]) = head;
}

// Emission, one launch: workgroups [0, kEmitBigBlocks) take the queued
// triangles with more than kBigCells cells, one triangle per workgroup at a
// time (lanes take rows, a block scan places them); the others take tiles of
// kTile triangles (256, 32 in small scenes, as a workgroup of the set-up): each lane writes its triangle's point offset (tile base +
// prefix within the tile), then the rows of the tile's small triangles are
// spread over the lanes; rows follow each other in emission order, so a scan of
// their cells places them.  Against a lane per triangle (up to 96 cells in one
// lane): 1.0M triangles 95 -> 77 us, 0.18M 62 -> 34 us.
constexpr unsigned kEmitBigBlocks = 1024;

template <int kTile>
__device__ __forceinline__ void emit_big(const EmitArgs& a, uint64_t* ws4) {
  const uint64_t nbig = *a.n_big;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (uint64_t b = blockIdx.x; b < nbig; b += kEmitBigBlocks) {
    const uint32_t t = a.big[b];
    const TriEmit& E = a.em[t];
    // the triangle's first point: the tile base plus the earlier counts in the tile
    const int64_t t0 = (int64_t)t - (int64_t)t % kTile;
    const int64_t u = t0 + threadIdx.x;
    const uint64_t cu = u < (int64_t)t ? a.counts[u] : 0u;
    uint64_t wsum = wave_sum(cu);
    if (lane == 0) ws4[wv] = wsum;
    __syncthreads();
    const uint64_t base = a.tile_base[t0 / kTile] + (ws4[0] + ws4[1]) + (ws4[2] + ws4[3]);
    __syncthreads();
    Lattice L;
    lattice_init(L, E.s1, E.t1, E.s2, E.t2);
    const int64_t jlo = E.jlo, jhi = E.jhi;  // rows with cells, found by the set-up
    uint64_t run = 0;
    for (int64_t j0 = jlo; j0 <= jhi; j0 += blockDim.x) {
      const int64_t j = j0 + threadIdx.x;
      int64_t lo = 1, hi = 0;
      if (j <= jhi) lattice_row(L, j, lo, hi);
      const uint64_t c = hi >= lo ? (uint64_t)(hi - lo + 1) : 0;
      uint64_t inc = wave_incl_scan(c);
      if (lane == 63) ws4[wv] = inc;
      __syncthreads();
      uint64_t before = 0, total = 0;
      for (int w = 0; w < 4; ++w) {
        if (w < wv) before += ws4[w];
        total += ws4[w];
      }
      const uint64_t start = base + run + before + inc - c;
      const uint32_t fj = (j == jlo ? F_JLO : 0u) | (j == jhi ? F_JHI : 0u);
      const uint64_t ri = base + (uint64_t)(j - jlo);
      if (a.rows && j <= jhi && ri < (uint64_t)a.cap)
        a.rows[ri] = RowEntry{(uint32_t)(start - base), (int16_t)lo, (int16_t)hi};
      for (int64_t i = lo; i <= hi; ++i) {
        uint64_t gi = start + (uint64_t)(i - lo);
        if (gi < (uint64_t)a.cap)
          write_head(a.points, gi, t, fj | (i == lo ? F_ILO : 0u) | (i == hi ? F_IHI : 0u), i, j);
      }
      run += total;
      __syncthreads();  // the wave sums are rewritten by the next pass
    }
  }
}

template <int kTile>
__global__ void __launch_bounds__(256) k_emit(EmitArgs a) {
  __shared__ uint64_t ws4[4];
  if (blockIdx.x < kEmitBigBlocks) {
    emit_big<kTile>(a, ws4);
    return;
  }
  __shared__ int4 l_st[kTile];         // s1, t1, s2, t2
  __shared__ int32_t l_jlo[kTile], l_jhi[kTile];
  __shared__ uint32_t l_rows[kTile];   // rows of the small triangles before this one
  __shared__ uint32_t l_first[kTile];  // its first point in the tile, and
  __shared__ uint32_t l_skip[kTile];   // the points of big triangles before it
  const int64_t tile = (int64_t)blockIdx.x - kEmitBigBlocks;
  const int64_t t0 = tile * kTile, t = t0 + threadIdx.x;
  const bool mine = (kTile == 256 || threadIdx.x < kTile) && t < a.nt;
  const uint32_t cnt = mine ? a.counts[t] : 0u;
  const uint64_t tbase = a.tile_base[tile];
  const uint32_t first = (uint32_t)block_excl_scan(cnt, ws4);  // kTile triangles of at most kCellCap points
  if (mine) a.offsets[t] = tbase + first;
  if (a.tris) {
    const uint64_t slot = wave_append(cnt > 0, a.n_tris);
    if (cnt > 0) a.tris[slot] = (uint32_t)t;
  }
  const bool small = cnt > 0 && cnt <= kBigCells;  // the big ones are queued by the set-up
  uint32_t nrows = 0;
  if (small) {
    const TriEmit& E = a.em[t];
    l_st[threadIdx.x] = make_int4(E.s1, E.t1, E.s2, E.t2);
    l_jlo[threadIdx.x] = E.jlo;
    l_jhi[threadIdx.x] = E.jhi;
    nrows = (uint32_t)(E.jhi - E.jlo + 1);
  }
  // one scan for both: rows (high word) and points of the big triangles (low word)
  const uint64_t sc = block_excl_scan(((uint64_t)nrows << 32) | (cnt > kBigCells ? cnt : 0u), ws4);
  if (kTile == 256 || threadIdx.x < kTile) {
    l_rows[threadIdx.x] = (uint32_t)(sc >> 32);
    l_skip[threadIdx.x] = (uint32_t)sc;
    l_first[threadIdx.x] = first;
  }
  const uint32_t total = (uint32_t)block_sum(nrows, ws4);
  uint32_t run = 0;  // points of the rows of earlier passes
  for (uint32_t k0 = 0; k0 < total; k0 += 256) {
    const uint32_t k = k0 + threadIdx.x;
    int q = 0;  // the last triangle whose rows begin at or before k: it has some
#pragma unroll
    for (int st = kTile / 2; st >= 1; st >>= 1)
      if (l_rows[q + st] <= k) q += st;
    int64_t j = 0, lo = 1, hi = 0;
    if (k < total) {
      const int4 st = l_st[q];
      Lattice L;
      lattice_init(L, st.x, st.y, st.z, st.w);
      j = (int64_t)l_jlo[q] + (int64_t)(k - l_rows[q]);
      lattice_row(L, j, lo, hi);
    }
    const uint32_t c = hi >= lo ? (uint32_t)(hi - lo + 1) : 0u;
    const uint32_t inc = (uint32_t)block_excl_scan(c, ws4);
    const uint32_t at = run + inc;  // rows follow each other in emission order, without the big triangles
    run += (uint32_t)block_sum(c, ws4);
    if (k >= total) continue;
    const uint32_t ti = (uint32_t)(t0 + q);
    const uint32_t fj = (j == l_jlo[q] ? F_JLO : 0u) | (j == l_jhi[q] ? F_JHI : 0u);
    const uint64_t start = tbase + at + l_skip[q];
    if (a.rows) {
      const uint64_t base = tbase + l_first[q], ri = base + (uint64_t)(j - l_jlo[q]);  // rows never outnumber points
      if (ri < (uint64_t)a.cap) a.rows[ri] = RowEntry{(uint32_t)(start - base), (int16_t)lo, (int16_t)hi};
    }
    for (int64_t i = lo; i <= hi; ++i) {
      const uint64_t gi = start + (uint64_t)(i - lo);
      if (gi < (uint64_t)a.cap)
        write_head(a.points, gi, ti, fj | (i == lo ? F_ILO : 0u) | (i == hi ? F_IHI : 0u), i, j);
    }
  }
}

// Splat rectangle of point (i, j): its lattice cell, extended by one cell
// beyond the end of its row (F_ILO / F_IHI) or of the lattice (F_JLO / F_JHI),
// with the corners projected except for the eye offset (x = cA - b*cC) and the
// range of their projected rows; `full` when a corner lies behind z_near/2.
__device__ __forceinline__ void splat_corners(const Rig& rg, const TriRec& T, int32_t i, int32_t j, uint32_t flags,
                                              float cA[4], float cC[4], float& ymn, float& ymx, bool& full) {
  const int32_t s0 = i - ((flags & F_ILO) ? 1 : 0), s1 = i + 1 + ((flags & F_IHI) ? 1 : 0);
  const int32_t t0 = j - ((flags & F_JLO) ? 1 : 0), t1 = j + 1 + ((flags & F_JHI) ? 1 : 0);
  const float zlim = 0.5f * rg.znear;
  ymn = ymx = 0.0f;
  full = false;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    float aa = ((float)((k & 1) ? s1 : s0) - 0.5f) / T.sx;
    float cc = ((float)((k & 2) ? t1 : t0) - 0.5f) / T.sy;
    float X = (T.p0x + aa * T.ux) + cc * T.wx;
    float Y = (T.p0y + aa * T.uy) + cc * T.wy;
    float Z = (T.p0z + aa * T.uz) + cc * T.wz;
    if (!(Z >= zlim)) full = true;
    float Yp;
    vertex_proj(rg, X, Y, Z, cA[k], cC[k], Yp);
    if (k == 0) { ymn = ymx = Yp; }
    else { ymn = Yp < ymn ? Yp : ymn; ymx = Yp > ymx ? Yp : ymx; }
  }
}

// Rows that splat_wave can write for a point in any view: the triangle's rows
// (guard band, the whole triangle above or below the view) met with the splat
// rectangle's rows `rows` (PointBox).  False when none.
__device__ __forceinline__ bool quilt_point_rows(int32_t H, const TriRec& T, int32_t rows, int32_t& r0, int32_t& r1) {
  if (!(fabsf(T.y0) < kGuard) || !(fabsf(T.y1) < kGuard) || !(fabsf(T.y2) < kGuard)) return false;
  const int32_t H8 = 256 * H;
  const int32_t qy0 = (int32_t)rintf(T.y0 * 256.0f), qy1 = (int32_t)rintf(T.y1 * 256.0f),
                qy2 = (int32_t)rintf(T.y2 * 256.0f);
  if ((qy0 < 0 && qy1 < 0 && qy2 < 0) || (qy0 > H8 && qy1 > H8 && qy2 > H8)) return false;
  const int32_t ymin = min(qy0, min(qy1, qy2)), ymax = max(qy0, max(qy1, qy2));
  r0 = max(0, -((128 - ymin) >> 8));
  r1 = min(H - 1, (ymax - 128) >> 8);
  if (rows != kAllRows) {
    r0 = max(r0, (int32_t)(int16_t)(rows & 0xFFFF));
    r1 = min(r1, (int32_t)(int16_t)((uint32_t)rows >> 16));
  }
  return r0 <= r1;
}

// Per point: UV at the cell centre and the two mip fetches (Eqs. 6-7); for the
// triangle-major splat and the quilt (kBox) also the point's splat rectangle
// (PointBox), for the quilt the pixel rows its splat can write; kPBR: the
// material fetches.  The plain form holds 46 VGPRs (8 waves per SIMD, for a
// kernel that waits on its texel gathers) instead of the 75 of all branches.
template <bool kBox, bool kPBR>
__global__ void __launch_bounds__(256) k_fetch(EmitArgs a) {
  const uint64_t npts = imin((int64_t)*a.n_points, a.cap);
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npts; p += stride) {
    uint2 head = *reinterpret_cast<const uint2*>(&a.points[p]);
    const uint32_t t = head.x & 0x0FFFFFFFu;
    const int64_t i = (int16_t)(head.y & 0xFFFFu), j = (int16_t)(head.y >> 16);
    const TriEmit& E = a.em[t];
    const int64_t S1 = E.s1, T1 = E.t1, S2 = E.s2, T2 = E.t2;
    const int64_t area2 = (S1 - 128) * (T2 - 128) - (T1 - 128) * (S2 - 128);
    int64_t cxq = 256 * i + 128, cyq = 256 * j + 128;
    int64_t w1 = (cxq - 128) * (T2 - 128) - (cyq - 128) * (S2 - 128);
    int64_t w2 = (S1 - 128) * (cyq - 128) - (T1 - 128) * (cxq - 128);
    // a zero-area lattice has no barycentrics: its points take vertex 0's UV
    float b1 = area2 != 0 ? (float)((double)w1 / (double)area2) : 0.0f;
    float b2 = area2 != 0 ? (float)((double)w2 / (double)area2) : 0.0f;
    float u = (E.uv0u + b1 * E.du1) + b2 * E.du2;
    float v = (E.uv0v + b1 * E.dv1) + b2 * E.dv2;
    const Item& it = a.items[E.item];
    const TexInfo& ti = it.texinfo[E.tex];
    uint2 tv;
    tv.x = trilinear(it.texels, ti, u, v, E.kmin);
    tv.y = E.kmax == E.kmin ? tv.x : trilinear(it.texels, ti, u, v, E.kmax);
    *reinterpret_cast<uint2*>(&a.points[p].tvmin) = tv;
    if constexpr (kBox) {
      const TriRec& T = a.rec[t];
      PointBox B;
      float ymn, ymx;
      bool full;
      splat_corners(it.rig, T, (int32_t)i, (int32_t)j, head.x >> 28, B.cA, B.cC, ymn, ymx, full);
      if (full) {
        B.rows = kAllRows;
      } else {
        // rows whose centres lie within 1/64 px of the corners' range, clamped
        // to [-1, H] (rows outside the view never matter)
        int32_t r0 = (int32_t)ceilf(clamp_big(ymn - 0.515625f)), r1 = (int32_t)floorf(clamp_big(ymx - 0.484375f));
        r0 = r0 < -1 ? -1 : (r0 > it.rig.H ? it.rig.H : r0);
        r1 = r1 < -1 ? -1 : (r1 > it.rig.H ? it.rig.H : r1);
        B.rows = (int32_t)((uint32_t)(uint16_t)(int16_t)r0 | ((uint32_t)(uint16_t)(int16_t)r1 << 16));
      }
      const float cs = (float)i / T.sx, ct = (float)j / T.sy;
      const float Zc = (T.p0z + cs * T.uz) + ct * T.wz;
      B.zc3 = (Zc * Zc) * Zc;
      B.tvmin = tv.x;
      B.tvmax = tv.y;
      a.pbox[p] = B;
      if (a.prows) {
        int32_t r0, r1;
        const uint32_t base = (uint32_t)E.item * (uint32_t)it.rig.H;
        a.prows[p] = quilt_point_rows(it.rig.H, T, B.rows, r0, r1) ? make_uint2(base + (uint32_t)r0, base + (uint32_t)r1)
                                                                   : make_uint2(~0u, ~0u);
      }
    }
    if constexpr (kPBR) {
      // physically based mode: normal map (RGBA8) and the R bytes of the
      // roughness and metallic maps, each at its own LOD pair
      const TriMat& M = a.tm[t];
      const TexInfo& tn = it.texinfo[M.texn];
      const TexInfo& tr = it.texinfo[M.texr];
      const TexInfo& tm = it.texinfo[M.texm];
      uint4 pm;
      pm.x = trilinear(it.texels, tn, u, v, M.kn0);
      pm.y = M.kn1 == M.kn0 ? pm.x : trilinear(it.texels, tn, u, v, M.kn1);
      const uint32_t r0 = trilinear(it.texels, tr, u, v, M.kr0) & 255u;
      const uint32_t r1 = M.kr1 == M.kr0 ? r0 : trilinear(it.texels, tr, u, v, M.kr1) & 255u;
      const uint32_t m0 = trilinear(it.texels, tm, u, v, M.km0) & 255u;
      const uint32_t m1 = M.km1 == M.km0 ? m0 : trilinear(it.texels, tm, u, v, M.km1) & 255u;
      pm.z = r0 | (r1 << 8) | (m0 << 16) | (m1 << 24);
      pm.w = 0u;
      a.pmat[p] = pm;
    }
  }
}

// ------------------------------------------------------------------ a3: splat

// An item table entry read by all active lanes of a wave from one address,
// moved to scalar registers word by word.
__device__ __forceinline__ Item load_uniform(const Item* p) {
  static_assert(sizeof(Item) % 4 == 0, "Item is a whole number of words");
  Item out;
  const int32_t* src = reinterpret_cast<const int32_t*>(p);
  int32_t* dst = reinterpret_cast<int32_t*>(&out);
#pragma unroll
  for (int k = 0; k < (int)(sizeof(Item) / 4); ++k) dst[k] = __builtin_amdgcn_readfirstlane(src[k]);
  return out;
}

// 64-bit depth-test update (relaxed, device scope); the key buffers are global
// memory, which lets the compiler issue a global rather than a flat atomic.
__device__ __forceinline__ void key_min(uint64_t* p, uint64_t v) {
  typedef __attribute__((address_space(1))) unsigned long long global_u64;
  __hip_atomic_fetch_min((global_u64*)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// 64-bit depth-test update of a key held in LDS (a quilt tile).
__device__ __forceinline__ void lds_key_min(uint64_t* p, uint64_t v) {
  typedef __attribute__((address_space(3))) unsigned long long lds_u64;
  __hip_atomic_fetch_min((lds_u64*)p, (unsigned long long)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One tile of the row-band quilt: views [r_lo, r_hi) and rows [y_lo, y_hi] of
// every view, all W columns, as keys[((r - r_lo) * rows + (y - y_lo)) * W + x]
// in LDS; `box` is the point's splat rectangle written at emission.
struct QuiltTile {
  uint64_t* keys;
  int32_t r_lo, r_hi, y_lo, y_hi, rows;
  const PointBox* box;
};

// Element i (wave-uniform) of a table that no kernel of the launch writes, as a
// scalar-cache read straight into a scalar register.
__device__ __forceinline__ float table_f32(const float* p, int i) {
  typedef const __attribute__((address_space(4))) float const_f32;
  return ((const_f32*)p)[i];
}

// Orders this wave's LDS accesses around it (its lanes exchange data there).
__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A wave's 64 points (one per lane) against views [r_begin, r_end) of their
// item's rig; `item` and the view range are wave-uniform, every lane of the
// wave calls, and lanes with `valid` false take part without a point.
//
// What bounds it: vector issue (the SIMDs issue vector instructions in 97 % of
// its cycles, in the quilt's tiles in all).  A (point, view) pair's splat box holds 1.7
// pixels on average but up to 4.4 in the slowest lane of 64, and of the box
// pixels 54 % lie inside the triangle and 29 % belong to the point, so a lane
// that carries its own pixels through the ray, the division, the ownership
// test, the colour and the key idles most of the time.  Three passes instead:
//   box pixels      per lane: 32-bit edge functions stepped over the box (the
//                   one part that walks at the pace of the largest box);
//   covered pixels  queued in LDS and taken 64 at a time, whichever lanes and
//                   views they came from: ray, depth, ownership, colour, key.
//                   The point's data come from its lane's registers
//                   (ds_bpermute), the view's from lanes that hold the tables;
//   owned pixels    (kPBR) queued once more, so that shading -- four fifths of
//                   the instructions there -- runs on full waves.
// A box of many pixels would hold its whole wave (one lane of a grazing
// triangle took 1.5 ms): all lanes walk it, 64 pixels at a time.
// Measured on a million-triangle frame (3.0M points, 48 views of 512 x 512)
// against one lane carrying each pixel to its key: 8.3e8 -> 4.8e8 vector
// instructions, 2.48 -> 1.17 ms (0.97 with the work items of k_splat and the
// statistics' lines).
// A queue entry is one word: lane (6 bits), x, y, and the view within a group
// of as many views as the remaining bits number (64 at most; 4 at 4096 x 4096).
//
// Edge functions: the triangle's vertices are taken in the order that makes
// its area positive for an eye in front of it, so dy, the tie rule (an edge
// owns its ties iff dy > 0, or dy == 0 and the third vertex lies below it) and
// the distance of the first row from each vertex do not depend on the view.
// A step of one pixel changes E by a multiple of 256, so E >> 8 carries its
// sign from pixel to pixel.  With spans up to kSmallSpan (124 pixels) E itself
// fits 32 bits and every factor 24, up to kLargeSpan (1562 pixels) E >> 8 does,
// in two parts.  A larger triangle, or one whose snapped area is not positive
// in this view, is walked by the whole wave with the exact 64-bit test
// (covered_wide).
//
// kQuilt: only the views and rows of tile *qt, keys in its LDS; the splat
// rectangle's corners, rows and cell-centre depth come from the point's
// PointBox (the same values, computed at emission).
//
// kHeld (a tile that leaves no LDS for the queues): up to 63 entries wait in
// one register, lane k's the k-th.  48 views of 600 x 512, the whole frame:
// 1764 us when a lane carried its point's pixels to their keys, 2489 when each
// covered pixel went through the passes by itself, 1294 with held entries; 192
// views of 640 x 480 5280, 8069 and 3809.  Where the LDS has room its queue is
// 2 to 4 % faster (48 views of 512 x 512: 1183 against 1208 us).
//
// Shaded tiles (no queue of owned pixels there): where coarse textures make
// points of many pixels, shading each owned pixel is dearer than shading each
// point.  A view in which the wave's large boxes (beyond kLaneSteps steps) hold
// kAheadPixels or more is shaded ahead, each lane its own point, and its pixels
// take the lane's colour; entries of views with and without such colours do not
// wait together.  48 views of 600 x 512, textures of 16 texels: 687 us with a
// lane's colour for all of its pixels, 836 shading each pixel, 660 so; of 8
// texels 1714, 1570 and 1191.  (From 96, 128 or 384 box pixels on: within 2 %;
// from 768: 3 to 15 % slower.)  The test costs 2 % where textures are fine.
constexpr int kSplatQueue = 191;        // entries: 63 waiting and 128 new ones at most
constexpr int32_t kLaneSteps = 8;       // steps of two pixels that a lane walks alone
constexpr int kAheadPixels = 192;       // box pixels of a wave in a view from which its points are shaded ahead
constexpr int kOwnQueue = 128;          // 63 waiting and 64 new ones
constexpr float kRound = 12582912.0f;    // 1.5 * 2^23: adding it rounds to an integer (ties to even) ...
constexpr int32_t kRoundBits = 0x4B400000;  // ... held in the sum's bits, offset by this
constexpr float kGuardQ8 = kGuard * 256.0f;
constexpr int32_t kSmallSpan = 31744;   // Q8: |E| <= 2 * 31744^2 + one step < 2^31
constexpr int32_t kLargeSpan = 400000;  // Q8: |E >> 8| <= 2 * 400000^2 / 256 + one step < 2^31

// a * b + c with 24-bit factors
__device__ __forceinline__ int32_t mad24(int32_t a, int32_t b, int32_t c) {
  int32_t d;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

__device__ __forceinline__ int32_t mul24(int32_t a, int32_t b) { return __mul24(a, b); }

__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

__device__ __forceinline__ float from_lane(int src4, float v) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src4, __float_as_int(v)));
}
__device__ __forceinline__ uint32_t from_lane(int src4, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_ds_bpermute(src4, (int)v);
}

// Is the centre of pixel (x, y) inside the Q8 triangle?  Exact for every
// vertex of the guard band.
__device__ __forceinline__ bool covered_wide(int32_t x, int32_t y, const int32_t qx[3], const int32_t qy[3]) {
  const int64_t a2 = (int64_t)(qx[1] - qx[0]) * (qy[2] - qy[0]) - (int64_t)(qy[1] - qy[0]) * (qx[2] - qx[0]);
  if (a2 == 0) return false;
  const int32_t px = 256 * x + 128, py = 256 * y + 128, s = a2 < 0 ? -1 : 1;
  bool in = true;
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int eb = e == 2 ? 0 : e + 1;
    const int32_t dx = s * (qx[eb] - qx[e]), dy = s * (qy[eb] - qy[e]);
    const int64_t E = (int64_t)dx * (py - qy[e]) - (int64_t)dy * (px - qx[e]);
    in = in && (E > 0 || (E == 0 && (dy > 0 || (dy == 0 && dx > 0))));
  }
  return in;
}

template <bool kPBR, bool kQuilt, bool kHeld>
__device__ __forceinline__ void splat_wave(const Item& item, bool valid, uint64_t p, const Point& pt, const TriRec& T,
                                           const float* tx, const float* ty, const SplatArgs& a, uint32_t* queue,
                                           uint2* own_queue, int r_begin, int r_end, uint32_t& written,
                                           const QuiltTile* qt = nullptr) {
  const Rig& rg = item.rig;
  const int lane = threadIdx.x & 63;
  const int32_t i = (int16_t)(pt.ij & 0xFFFFu), j = (int16_t)(pt.ij >> 16);
  const int32_t H8 = 256 * rg.H;
  // view-independent vertex rows (guard band on y) and triangle row range
  bool alive = valid && fabsf(T.y0) < kGuard && fabsf(T.y1) < kGuard && fabsf(T.y2) < kGuard;
  const int32_t qy[3] = {(int32_t)rintf(T.y0 * 256.0f), (int32_t)rintf(T.y2 * 256.0f), (int32_t)rintf(T.y1 * 256.0f)};
  const int32_t ymin = min(qy[0], min(qy[1], qy[2])), ymax = max(qy[0], max(qy[1], qy[2]));
  alive = alive && ymax >= 0 && ymin <= H8;
  int32_t by0 = max(0, (ymin + 127) >> 8), by1 = min(rg.H - 1, (ymax - 128) >> 8);
  // splat box corners (row-end extended cell), projected except for the eye offset
  float cA[4], cC[4];
  bool full;
  if constexpr (kQuilt) {
    // the stored rows are clamped to [-1, H], which leaves their intersection
    // with the triangle's rows (inside [0, H-1]) unchanged or empty as before
    const PointBox& B = *qt->box;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      cA[k] = B.cA[k];
      cC[k] = B.cC[k];
    }
    full = B.rows == kAllRows;
    if (!full) {
      by0 = max((int32_t)(int16_t)(B.rows & 0xFFFF), by0);
      by1 = min((int32_t)(int16_t)((uint32_t)B.rows >> 16), by1);
    }
    by0 = max(by0, qt->y_lo);
    by1 = min(by1, qt->y_hi);
  } else {
    float ymn, ymx;
    splat_corners(rg, T, i, j, pt.tri_flags >> 28, cA, cC, ymn, ymx, full);
    if (!full) {
      by0 = max((int32_t)ceilf(clamp_big(ymn - 0.515625f)), by0);
      by1 = min((int32_t)floorf(clamp_big(ymx - 0.484375f)), by1);
    }
  }
  if (full) {  // no box limit: columns -2^29 .. 2^29 in every view
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      cA[k] = (k & 1) ? 0x1p29f : -0x1p29f;
      cC[k] = 0.0f;
    }
  }
  alive = alive && by0 <= by1;
  if (!__builtin_amdgcn_ballot_w64(alive)) return;
  // cell-centre terms of Eqs. 8-9
  float pcx = 0.0f, pcy = 0.0f, zc;  // zc: the centre's depth (kPBR) or its cube
  if (kQuilt && !kPBR) {
    zc = qt->box->zc3;
  } else {
    const float cs = (float)i / T.sx, ct = (float)j / T.sy;
    zc = (T.p0z + cs * T.uz) + ct * T.wz;
    if constexpr (kPBR) {
      pcx = (T.p0x + cs * T.ux) + ct * T.wx;
      pcy = (T.p0y + cs * T.uy) + ct * T.wy;
    } else {
      zc = (zc * zc) * zc;
    }
  }
  const float acell = 1.0f / (T.sx * T.sy);
  const float p0y2 = T.p0y * T.p0y, p0z2 = T.p0z * T.p0z;
  // lattice cell of the point; a NaN bound (an end of its row or lattice) excludes nothing
  const uint32_t flags = pt.tri_flags >> 28;
  const float kNone = __uint_as_float(0x7FC00000u);
  const float s_lo = (flags & F_ILO) ? kNone : (float)i, s_hi = (flags & F_IHI) ? kNone : (float)(i + 1);
  const float t_lo = (flags & F_JLO) ? kNone : (float)j, t_hi = (flags & F_JHI) ? kNone : (float)(j + 1);
  // edges 0-1, 1-2, 2-0 of the vertices 0, 2, 1 of the record; in 1/256 px (an exact scaling)
  const float va[3] = {T.a0 * 256.0f, T.a2 * 256.0f, T.a1 * 256.0f};
  const float vc[3] = {T.c0 * 256.0f, T.c2 * 256.0f, T.c1 * 256.0f};
  int32_t ndy[3], py[3], tie[3];
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const int eb = e == 2 ? 0 : e + 1, ec = eb == 2 ? 0 : eb + 1;
    ndy[e] = qy[e] - qy[eb];
    py[e] = 256 * by0 + 128 - qy[e];
    tie[e] = (ndy[e] < 0 || (ndy[e] == 0 && qy[ec] > qy[e])) ? 0 : -1;
  }
  const uint64_t tall_m = __builtin_amdgcn_ballot_w64(ymax - ymin > kSmallSpan);
  const uint64_t huge_m = __builtin_amdgcn_ballot_w64(ymax - ymin > kLargeSpan);
  const float x_last = (float)(rg.W - 1);
  const int32_t tsum = tie[0] + tie[1] + tie[2];
  // Facing and guard-band tests that hold for every eye are settled once: the
  // plane distance, its square, the eye distance and each projected x are
  // monotone in the eye offset (rounding keeps order), so both ends decide.
  bool safe;
  {
    const float d0 = T.h - T.nx * rg.eye_lo, d1 = T.h - T.nx * rg.eye_hi;
    const float dm = fminf(fabsf(d0), fabsf(d1));
    const float e0 = T.p0x - rg.eye_lo, e1 = T.p0x - rg.eye_hi;
    const float d2 = fmaxf((e0 * e0 + p0y2) + p0z2, (e1 * e1 + p0y2) + p0z2);
    safe = d0 < 0.0f && d1 < 0.0f && dm * dm >= d2 * 0x1p-16f;
#pragma unroll
    for (int k = 0; k < 3; ++k)
      safe = safe && fabsf(va[k] - rg.eye_lo * vc[k]) < kGuardQ8 && fabsf(va[k] - rg.eye_hi * vc[k]) < kGuardQ8;
  }
  const uint64_t alive_m = __builtin_amdgcn_ballot_w64(alive);
  const bool all_safe = (alive_m & ~__builtin_amdgcn_ballot_w64(safe)) == 0;
  const int32_t nrows = by1 - by0 + 1;
  // queue entries: lane | x << 6 | y << ysh | view of the group << rsh
  const int xb = rg.W > 1 ? 32 - __builtin_clz((uint32_t)rg.W - 1u) : 0, yb = rg.H > 1 ? 32 - __builtin_clz((uint32_t)rg.H - 1u) : 0;
  const int ysh = 6 + xb, rsh = 6 + xb + yb;
  const uint32_t xm = (1u << xb) - 1u, ym = (1u << yb) - 1u;
  const int group = rsh <= 26 ? 64 : 1 << (32 - rsh);
  const bool rowmajor = item.key_layout != 0;
  uint32_t qn = 0, on_n = 0;  // waiting entries: covered pixels; owned pixels (kPBR)
  uint32_t held = 0;          // kHeld: lane k's waiting entry, k < qn
  constexpr bool kAhead = kPBR && kQuilt;
  uint32_t ahead = 0;         // kAhead: 1 if this view's colours are in col_l, lane k's of point k
  uint32_t col_l = 0;
  float eye_l = 0.0f, ks_l = 0.0f;  // eye offset and lens shift of view g0 + lane
  int g0 = r_begin;

  // Colour (Eqs. 8-9; kPBR: shaded) of owned pixel e at depth Z, and its key.  kAhead: the view's colours may be there
  // already; `first` puts them there, for entries of no pixel.
  auto emit_key = [&](uint32_t e, float Z, bool on, float b, float nx, float delta, bool first, bool there) {
    const int src = (int)((e & 63u) << 2);
    const uint32_t x = (e >> 6) & xm, y = (e >> ysh) & ym, rr = e >> rsh;
    auto tile_key = [&](uint32_t col) {
      lds_key_min(qt->keys + (((g0 - qt->r_lo + (int)rr) * qt->rows + ((int)y - qt->y_lo)) * rg.W + (int)x),
                  ((uint64_t)__float_as_uint(Z) << 32) | col);
    };
    if (kAhead && there) {
      const uint32_t col = from_lane(src, col_l);
      if (on) tile_key(col);
      return;
    }
    const float ac = from_lane(src, acell), ruv = from_lane(src, T.ruv);
    const float smin = from_lane(src, T.smin), smax = from_lane(src, T.smax), irange = from_lane(src, T.irange);
    const uint32_t lo = from_lane(src, pt.tvmin), hi = from_lane(src, pt.tvmax);
    float zc3 = from_lane(src, zc);
    F3 ng{nx, 0.0f, 0.0f}, pc{0.0f, 0.0f, zc3};
    uint32_t tri = 0;
    uint64_t pp = 0;
    if constexpr (kPBR) {
      ng.y = from_lane(src, T.ny);
      ng.z = from_lane(src, T.nz);
      pc.x = from_lane(src, pcx);
      pc.y = from_lane(src, pcy);
      zc3 = (zc3 * zc3) * zc3;
      tri = from_lane(src, pt.tri_flags) & 0x0FFFFFFFu;
      pp = (uint64_t)from_lane(src, (uint32_t)p) | ((uint64_t)from_lane(src, (uint32_t)(p >> 32)) << 32);
    }
    if (!on) return;
    const float ad = fabsf(delta);
    const float Ar = zc3 / (rg.fxfy * ad);
    const float vse = ac < Ar ? ruv * Ar : ac * ruv;
    const float vs = vse < smin ? smin : (vse > smax ? smax : vse);
    const float tau = (vs - smin) * irange;
    int32_t tq = (int32_t)floorf(tau * 256.0f + 0.5f);
    tq = tq < 0 ? 0 : (tq > 256 ? 256 : tq);
    const uint32_t wa = (uint32_t)(256 - tq), wz = (uint32_t)tq;
    auto lerp_even = [&](uint32_t u, uint32_t v) {  // bytes 0 and 2 of each word
      return (((u & 0x00FF00FFu) * wa + (v & 0x00FF00FFu) * wz + 0x00800080u) >> 8) & 0x00FF00FFu;
    };
    uint32_t col = lerp_even(lo, hi) | (lerp_even(lo >> 8, hi >> 8) << 8);
    if constexpr (kPBR) {
      // the normal map and the roughness / metallic bytes take the same tau
      const TriMat& M = a.tm[tri];
      const uint4 pm = a.pmat[pp];
      const uint32_t nrm = lerp_even(pm.x, pm.y) | (lerp_even(pm.x >> 8, pm.y >> 8) << 8);
      const uint32_t rq = ((pm.z & 255u) * wa + ((pm.z >> 8) & 255u) * wz + 128u) >> 8;
      const uint32_t mq = (((pm.z >> 16) & 255u) * wa + (pm.z >> 24) * wz + 128u) >> 8;
      col = shade_splat(a.sh, ng, F3{M.tx, M.ty, M.tz}, F3{M.bx, M.by, M.bz}, pc, b, col, nrm, rq, mq);
    }
    const uint64_t key = ((uint64_t)__float_as_uint(Z) << 32) | col;
    if constexpr (kQuilt) {
      if (kAhead && first) col_l = col;
      else tile_key(col);
    } else {
      const uint32_t r = (uint32_t)g0 + rr;
      const uint32_t row = rowmajor ? y * (uint32_t)rg.n_views + r : r * (uint32_t)rg.H + y;
      key_min(item.keys + ((uint64_t)row * (uint32_t)rg.W + x), key);
    }
  };

  auto emit_queued = [&](uint2 q, bool on) {
    const float b = from_lane((int)((q.x >> rsh) << 2), eye_l), nx = from_lane((int)((q.x & 63u) << 2), T.nx);
    emit_key(q.x, __uint_as_float(q.y), on, b, nx, from_lane((int)((q.x & 63u) << 2), T.h) - nx * b, false, false);
  };

  // Covered pixel e of each lane of mask `on`: ray hit, depth, ownership.
  auto take = [&](uint32_t e, uint64_t on, bool there) {
    const int src = (int)((e & 63u) << 2);
    const uint32_t x = (e >> 6) & xm, y = (e >> ysh) & ym;
    const int vsrc = (int)((e >> rsh) << 2);
    const float b = from_lane(vsrc, eye_l);
    const float rx = tx[x] - from_lane(vsrc, ks_l), ry = ty[y];
    const float nx = from_lane(src, T.nx);
    const float delta = from_lane(src, T.h) - nx * b;
    const float den = (nx * rx + from_lane(src, T.ny) * ry) + from_lane(src, T.nz);
    const float ux = from_lane(src, T.ux), wx = from_lane(src, T.wx);
    const float bp = b - from_lane(src, T.p0x);
    const float cu = ux * bp - from_lane(src, T.cu0);
    const float cw = wx * bp - from_lane(src, T.cw0);
    const float ur = (ux * rx + from_lane(src, T.uy) * ry) + from_lane(src, T.uz);
    const float wr = (wx * rx + from_lane(src, T.wy) * ry) + from_lane(src, T.wz);
    const float Z = delta / den;
    const float sv = from_lane(src, T.sx) * (Z * ur + cu) + 0.5f;
    const float tv = from_lane(src, T.sy) * (Z * wr + cw) + 0.5f;
    const uint64_t m = on & __builtin_amdgcn_ballot_w64(Z > 0.0f) & __builtin_amdgcn_ballot_w64(Z < INFINITY) &
                       ~__builtin_amdgcn_ballot_w64(sv < from_lane(src, s_lo)) &
                       ~__builtin_amdgcn_ballot_w64(sv >= from_lane(src, s_hi)) &
                       ~__builtin_amdgcn_ballot_w64(tv < from_lane(src, t_lo)) &
                       ~__builtin_amdgcn_ballot_w64(tv >= from_lane(src, t_hi));
    if (!m) return;
    const bool own = __builtin_amdgcn_inverse_ballot_w64(m);
    written += (uint32_t)__builtin_popcountll(m);
    if (kPBR && own_queue) {
      if (own) own_queue[on_n + lanes_below(m)] = make_uint2(e, __float_as_uint(Z));
      on_n += (uint32_t)__builtin_popcountll(m);
      if (on_n >= 64) {
        on_n -= 64;
        wave_sync_lds();
        const uint2 q = own_queue[on_n + lane];
        wave_sync_lds();
        emit_queued(q, true);
      }
    } else {
      emit_key(e, Z, own, b, nx, delta, false, there);
    }
  };

  // kHeld: the lanes of m send their entries to lanes qn, qn + 1, .. (the others send theirs to the lanes after
  // those, so that the whole wave exchanges a permutation, which needs no LDS storage).
  auto hold = [&](uint32_t e, uint64_t m) {
    const uint32_t n = (uint32_t)__builtin_popcountll(m), below = lanes_below(m);
    const uint32_t to = qn + (__builtin_amdgcn_inverse_ballot_w64(m) ? below : n + (uint32_t)lane - below);
    const uint32_t got = (uint32_t)__builtin_amdgcn_ds_permute((int)((to & 63u) << 2), (int)e);
    held = (uint32_t)lane >= qn ? got : held;
    qn = (uint32_t)__builtin_amdgcn_readfirstlane((int)(qn + n));
    if (qn >= 64) {
      if (kAhead && ahead) take(held, ~0ull, true);
      else take(held, ~0ull, false);
      held = got;
      qn -= 64;
    }
  };

  // Pixel e of each lane of mask m0 and the next one of m1 are covered: queued, and taken 64 at a time.
  auto push = [&](uint32_t e, uint64_t m0, uint64_t m1) {
    if (!(m0 | m1)) return;
    if constexpr (kHeld) {
      if (m0) hold(e, m0);
      if (m1) hold(e + 64u, m1);
      return;
    }
    const uint32_t n0 = (uint32_t)__builtin_popcountll(m0);
    if (__builtin_amdgcn_inverse_ballot_w64(m0)) queue[qn + lanes_below(m0)] = e;
    if (__builtin_amdgcn_inverse_ballot_w64(m1)) queue[qn + n0 + lanes_below(m1)] = e + 64u;
    // the same in every lane, which the compiler does not see through the loops around
    qn = (uint32_t)__builtin_amdgcn_readfirstlane((int)(qn + n0 + (uint32_t)__builtin_popcountll(m1)));
    while (qn >= 64) {
      qn -= 64;
      wave_sync_lds();
      const uint32_t te = queue[qn + lane];
      wave_sync_lds();
      if (kAhead && ahead) take(te, ~0ull, true);
      else take(te, ~0ull, false);
    }
  };

  for (int next; g0 < r_end; g0 = kAhead ? next : g0 + group) {
    const int g1 = min(r_end, g0 + group);
    next = g1;
    const int rl = min(g0 + lane, r_end - 1);
    eye_l = rg.eye[rl];
    ks_l = rg.kshift[rl];
    float b_next = table_f32(rg.eye, g0);  // the next view's eye offset, one iteration ahead
    for (int r = g0; r < g1; ++r) {
      const float b = b_next;
      if (r + 1 < g1) b_next = table_f32(rg.eye, r + 1);
      uint64_t act = alive_m;
      if (!all_safe) act &= __builtin_amdgcn_ballot_w64(faces_eye(T.p0x, p0y2, p0z2, T.h - T.nx * b, b));
      // splat box columns first: empty for about a third of the (point, view) pairs
      const float c0 = cA[0] - b * cC[0], c1 = cA[1] - b * cC[1], c2 = cA[2] - b * cC[2], c3 = cA[3] - b * cC[3];
      const float xmn = fminf(fminf(c0, c1), fminf(c2, c3)), xmx = fmaxf(fmaxf(c0, c1), fmaxf(c2, c3));
      int32_t bx0 = (int32_t)ceilf(__builtin_amdgcn_fmed3f(xmn - 0.515625f, 0.0f, 8192.0f));
      int32_t bx1 = (int32_t)floorf(__builtin_amdgcn_fmed3f(xmx - 0.484375f, -1.0f, x_last));
      act &= __builtin_amdgcn_ballot_w64(bx0 <= bx1);
      if (!act) continue;
      // Q8 vertices, rounded to integers in the low mantissa bits (offset by kRoundBits): exact up to 2^22, that
      // is 16384 px; beyond, still monotone, so far off every view (at most 4096 px wide) as before
      const float x0 = va[0] - b * vc[0], x1 = va[1] - b * vc[1], x2 = va[2] - b * vc[2];
      if (!all_safe)
        act &= __builtin_amdgcn_ballot_w64(fabsf(x0) < kGuardQ8 && fabsf(x1) < kGuardQ8 && fabsf(x2) < kGuardQ8);
      const int32_t q0 = __float_as_int(x0 + kRound), q1 = __float_as_int(x1 + kRound), q2 = __float_as_int(x2 + kRound);
      const int32_t xmin = min(q0, min(q1, q2)), xmax = max(q0, max(q1, q2));
      bx0 = max(bx0, (xmin - (kRoundBits - 127)) >> 8);
      bx1 = min(bx1, (xmax - (kRoundBits + 128)) >> 8);
      const int32_t w = bx1 - bx0 + 1;
      act &= __builtin_amdgcn_ballot_w64(w > 0);
      const int32_t pxq = 256 * bx0 + (128 + kRoundBits);
      const int32_t dx0 = q1 - q0, dx1 = q2 - q1, dx2 = q0 - q2;
      // edge functions at (bx0, by0), minus one where the edge does not own its ties: covered iff none is negative
      int32_t R0 = mad24(ndy[0], pxq - q0, mad24(dx0, py[0], tie[0]));
      int32_t R1 = mad24(ndy[1], pxq - q1, mad24(dx1, py[1], tie[1]));
      int32_t R2 = mad24(ndy[2], pxq - q2, mad24(dx2, py[2], tie[2]));
      // their sum is the doubled area (plus tsum) at every pixel
      uint64_t wide = __builtin_amdgcn_ballot_w64((int32_t)((uint32_t)R0 + (uint32_t)R1 + (uint32_t)R2) <= tsum);
      R0 >>= 8;
      R1 >>= 8;
      R2 >>= 8;
      const uint64_t large = act & (tall_m | __builtin_amdgcn_ballot_w64(xmax - xmin > kSmallSpan));
      if (large) {
        // E >> 8 from the whole and the fractional pixels of the distances
        auto edge = [&](int32_t q, int32_t dx, int32_t nd, int32_t pye, int32_t te) {
          const int32_t px = pxq - q;
          return mad24(nd, (px + 128) >> 8, mul24(dx, (pye + 128) >> 8)) +
                 (mad24(nd, ((px + 128) & 255) - 128, mad24(dx, ((pye + 128) & 255) - 128, te)) >> 8);
        };
        const bool lg = __builtin_amdgcn_inverse_ballot_w64(large);
        const int32_t L0 = edge(q0, dx0, ndy[0], py[0], tie[0]), L1 = edge(q1, dx1, ndy[1], py[1], tie[1]),
                      L2 = edge(q2, dx2, ndy[2], py[2], tie[2]);
        R0 = lg ? L0 : R0;
        R1 = lg ? L1 : R1;
        R2 = lg ? L2 : R2;
        // not positive here includes every triangle whose area is not
        wide = (wide & ~large) | (large & __builtin_amdgcn_ballot_w64((int32_t)((uint32_t)L0 + (uint32_t)L1 + (uint32_t)L2) <= 0)) |
               (large & (huge_m | __builtin_amdgcn_ballot_w64(xmax - xmin > kLargeSpan)));
      }
      // Lanes walk their own boxes, two pixels of a row at a time.  Boxes beyond
      // some number of steps (and wide triangles) are left to the whole wave, 64
      // pixels at a time: a step costs the wave a quarter of such a box, so the
      // limit follows how many boxes exceed it.
      const int32_t steps = __mul24((w + 1) >> 1, nrows);
      uint64_t over = act & __builtin_amdgcn_ballot_w64(steps > kLaneSteps);
      uint32_t many = 0;
      if (over) {
        const uint64_t over4 = over & __builtin_amdgcn_ballot_w64(steps > 4 * kLaneSteps);
        if constexpr (kAhead) {
          const int32_t px = 2 * kLaneSteps * (int32_t)(__builtin_popcountll(over) + 3 * __builtin_popcountll(over4));
          if (px >= kAheadPixels || (over4 & __builtin_amdgcn_ballot_w64(steps > kAheadPixels / 2))) many = 1;
        }
        if (__builtin_popcountll(over) - __builtin_popcountll(over4) > 3 * kLaneSteps / 4) over = over4;
      }
      if constexpr (kAhead) {
        if (qn && (many | ahead)) {  // what waits has the colours of its own views: this one begins the next group
          next = r;
          break;
        }
        ahead = (uint32_t)__builtin_amdgcn_readfirstlane((int)many);
        if (ahead)
          emit_key((uint32_t)lane | ((uint32_t)(r - g0) << rsh), 0.0f, __builtin_amdgcn_inverse_ballot_w64(act), b, T.nx,
                   T.h - T.nx * b, true, false);
      }
      uint64_t heavy = (act & wide) | over;
      const uint32_t e0 = (uint32_t)((bx0 << 6) + (int32_t)((uint32_t)lane | ((uint32_t)by0 << ysh))) + ((uint32_t)(r - g0) << rsh);
      int32_t rem = (__builtin_amdgcn_inverse_ballot_w64(act & ~heavy) ? steps : 0) - 1;  // steps after this one
      if (__builtin_amdgcn_ballot_w64(rem >= 0)) {
        int32_t E0 = R0, E1 = R1, E2 = R2, cx = rem >= 0 ? w - 2 : 1 << 20;  // columns after the pair (none wraps that has no box)
        uint32_t e = e0;
        for (;;) {
          const uint64_t m0 = __builtin_amdgcn_ballot_w64((E0 | E1 | E2 | rem) >= 0);
          E0 += ndy[0];
          E1 += ndy[1];
          E2 += ndy[2];
          push(e, m0, __builtin_amdgcn_ballot_w64((E0 | E1 | E2 | rem | cx) >= 0));
          rem -= 1;
          if (!__builtin_amdgcn_ballot_w64(rem >= 0)) break;
          cx -= 2;
          e += 128u;
          E0 += ndy[0];
          E1 += ndy[1];
          E2 += ndy[2];
          if (cx < -1) {  // the next row of the box
            cx = w - 2;
            e += (1u << ysh) - (((uint32_t)w + 1u) >> 1 << 7);
            E0 = R0 += dx0;
            E1 = R1 += dx1;
            E2 = R2 += dx2;
          }
        }
      }
      while (heavy) {
        const int32_t hl = (int32_t)__builtin_ctzll(heavy);
        const bool exact = (wide >> hl) & 1;
        heavy &= heavy - 1;
        const int32_t hw = __builtin_amdgcn_readlane(w, hl), hn = hw * __builtin_amdgcn_readlane(nrows, hl);
        const uint32_t he = (uint32_t)__builtin_amdgcn_readlane((int)e0, hl);
        int32_t qx[3], qyw[3];
        const int32_t wy = 256 * __builtin_amdgcn_readlane(by0, hl) + 128;
        if (exact) {
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            const float ha = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(va[k]), hl));
            const float hc = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(vc[k]), hl));
            qx[k] = (int32_t)rintf(ha - b * hc);
            qyw[k] = wy - __builtin_amdgcn_readlane(py[k], hl);
          }
        }
        const int32_t H0 = __builtin_amdgcn_readlane(R0, hl), H1 = __builtin_amdgcn_readlane(R1, hl), H2 = __builtin_amdgcn_readlane(R2, hl);
        const int32_t n0 = __builtin_amdgcn_readlane(ndy[0], hl), n1 = __builtin_amdgcn_readlane(ndy[1], hl), n2 = __builtin_amdgcn_readlane(ndy[2], hl);
        const int32_t d0 = __builtin_amdgcn_readlane(dx0, hl), d1 = __builtin_amdgcn_readlane(dx1, hl), d2 = __builtin_amdgcn_readlane(dx2, hl);
        const float inv = 1.0f / (float)hw;
        for (int32_t k0 = 0; k0 < hn; k0 += 64) {
          // pixel k of the box: row k / hw by the float reciprocal (k < 2^24, off by one at most)
          const int32_t k = k0 + lane;
          int32_t yq = (int32_t)((float)k * inv), xq = k - yq * hw;
          if (xq < 0) { yq -= 1; xq += hw; }
          else if (xq >= hw) { yq += 1; xq -= hw; }
          const uint32_t e = he + ((uint32_t)xq << 6) + ((uint32_t)yq << ysh);
          bool in;
          if (exact)
            in = covered_wide((int32_t)((e >> 6) & xm), (int32_t)((e >> ysh) & ym), qx, qyw);
          else
            in = ((H0 + mul24(n0, xq) + mul24(d0, yq)) | (H1 + mul24(n1, xq) + mul24(d1, yq)) |
                  (H2 + mul24(n2, xq) + mul24(d2, yq))) >= 0;
          push(e, __builtin_amdgcn_ballot_w64(k < hn && in), 0);
        }
      }
    }
    // what waits goes before the group's tables are replaced
    if (qn) {
      wave_sync_lds();
      const uint32_t te = (uint32_t)lane < qn ? (kHeld ? held : queue[lane]) : 0u;
      wave_sync_lds();
      const uint64_t on = ~(~0ull << qn);
      qn = 0;
      if (kAhead && ahead) take(te, on, true);
      else take(te, on, false);
    }
    if (kPBR && on_n) {
      wave_sync_lds();
      const bool on = (uint32_t)lane < on_n;
      const uint2 q = on ? own_queue[lane] : make_uint2(0u, 0u);
      wave_sync_lds();
      on_n = 0;
      emit_queued(q, on);
    }
  }
}

// kMulti: points of several items (a batch); otherwise every point belongs to
// items[0] and the item is read once.  kPBR: shaded colours.
// Work items are 64 consecutive points (a chunk) and the views, or a part of
// the views when the frame has fewer than 2 kFillItems chunks: half of them, or
// as few as make kFillItems items (a frame of 20 thousand points is 315 waves
// of up to V dependent steps otherwise; the point set-up is repeated for each
// part).  Waves draw items from kWorkQueues counters, each wave from one of
// them: with a fixed stride the chip waits for its slowest waves for a third of
// the launch, as items of 60 us at the median take 190 at the 99th and 410 at
// the last percentile; one counter for all hands out only some 60 items in a
// microsecond.  Measured (frames of 0.65M points, 25 views of 317 x 253, and
// 3.0M points, 48 views of 512 x 512): all views 440 and 1505 us, this rule 420
// and 1455, twice as many items 438 and 1455.
// The parts follow each other, all chunks in one part of the views before the
// next (in a batch, one item's after the other's), and there are as many as the
// keys of all views take kReachKeys (192 MiB, so that a part's updates are
// resolved in the 256 MiB last-level cache), a part's views rounded up: 48 views
// of 1024 x 1024 in one part 4.15 ms, in two 3.39.  Large views: 5 of 4096 x 4096
// in parts of two views (256 MiB of keys) 5.51 ms, of one 6.02, since each part
// repeats the points' set-up.
constexpr uint64_t kReachKeys = 24ull << 20;
constexpr uint32_t kFillItems = 32768;

template <bool kMulti, bool kPBR>
__global__ void __launch_bounds__(256) k_splat(SplatArgs a) {
  if (a.gate && *a.gate == 0) return;
  extern __shared__ float ray_tab[];  // W column slopes, then H row slopes
  __shared__ uint32_t queues[4][kSplatQueue];
  __shared__ uint2 own_queues[kPBR ? 4 : 1][kPBR ? kOwnQueue : 1];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t queues_n = min((uint32_t)kWorkQueues, gridDim.x * 4);  // every queue has a wave
  const uint32_t wq = (blockIdx.x * 4 + (uint32_t)wv) % queues_n;
  uint32_t* const next = reinterpret_cast<uint32_t*>(a.stats + kStatLines + LINE_WORDS * wq + LINE_NEXT);
  auto draw = [&]() {  // the next item of this wave's queue
    uint32_t k = 0;
    if (lane == 0) k = atomicAdd(next, 1u);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)k) * queues_n + wq;
  };
  uint32_t c = draw();
  const Rig& trg = a.table_rig;
  float* tx = ray_tab;
  float* ty = ray_tab + trg.W;
  for (int k = threadIdx.x; k < trg.W; k += blockDim.x) tx[k] = ((float)k + 0.5f - trg.cx) / trg.fx;
  for (int k = threadIdx.x; k < trg.H; k += blockDim.x) ty[k] = ((float)k + 0.5f - trg.cy) / trg.fy;
  __syncthreads();
  const uint64_t npts = imin((int64_t)*a.n_points, a.cap);
  uint32_t* const queue = queues[wv];
  uint2* const own_queue = kPBR ? own_queues[wv] : nullptr;
  const Item it0 = load_uniform(a.items);
  uint32_t written = 0;
  const uint32_t chunks = (uint32_t)((npts + 63) >> 6), V = (uint32_t)trg.n_views;
  const uint32_t fill = chunks >= 2 * kFillItems || chunks == 0 ? 1u : max(2u, (kFillItems + chunks - 1) / chunks);
  const uint32_t reach = (uint32_t)(((uint64_t)V * (uint32_t)trg.W * (uint32_t)trg.H + kReachKeys - 1) / kReachKeys);
  const uint32_t want = max(1u, min(min(V, max(fill, reach)), 0x7fffffffu / max(1u, chunks)));  // items in 31 bits
  const uint32_t per = (V + want - 1) / want, parts = (V + per - 1) / per;  // views per item, items per chunk
  for (; c < chunks * parts; c = draw()) {
    const uint32_t part = c / chunks, chunk = c - part * chunks, r0 = part * per, r1 = min(V, r0 + per);
    uint64_t p = (uint64_t)chunk * 64 + (uint64_t)lane;
    const bool valid = p < npts;
    p = valid ? p : npts - 1;
    const Point pt = a.points[p];
    const uint32_t tri = pt.tri_flags & 0x0FFFFFFFu;
    if (!kMulti) {
      const TriRec T = a.rec[tri];
      splat_wave<kPBR, false, false>(it0, valid, p, pt, T, tx, ty, a, queue, own_queue, (int)r0, (int)r1, written);
      continue;
    }
    // points of one wave nearly always belong to one item: take the items one at
    // a time, each pass with a uniform item.  The loop runs on a ballot mask, so
    // its trip count is the same in every lane and the body stays inside it.
    // Only the record's item is read before the loop (the whole record inside).
    const int32_t my = a.rec[tri].item;
    uint64_t todo = __builtin_amdgcn_ballot_w64(valid);
    while (todo) {
      const int32_t cur = __builtin_amdgcn_readlane(my, (int32_t)__builtin_ctzll(todo));
      const bool mine = valid && my == cur;
      const Item it = load_uniform(a.items + cur);
      const TriRec T = a.rec[tri];
      splat_wave<kPBR, false, false>(it, mine, p, pt, T, tx, ty, a, queue, own_queue, (int)r0, (int)r1, written);
      todo &= ~__builtin_amdgcn_ballot_w64(mine);
    }
  }
  if (lane == 0) line_add(a.stats, LINE_WRITTEN, written);
}

// ------------------------------------------------------------------ a3: splat, row-band quilt
//
// The keys of one tile -- q_rows pixel rows of q_views views, all W columns --
// stay in LDS while every point whose splat reaches those rows is splatted
// into them (64-bit ds_min), and the finished tile is written out as the
// views' RGBA8 (+ depth): the key buffer in HBM is neither updated nor
// resolved.  The views differ only by a horizontal eye offset (Sec. 3.2), so a
// point's pixel rows are the same in every view and each point is binned once
// per frame, into every band of q_rows rows that its splat can reach (in a
// batch, the bands of its own item).  A workgroup takes one tile; tiles are
// launched by decreasing band size.  Workgroups have 1024 threads (16 waves,
// one tile per CU), or 512 when two tiles fit the CU's LDS.

constexpr int kQChunk = 4096;  // points per workgroup pass in the band kernels

// Band (over all items) of stacked row g = item * H + row.
__device__ __forceinline__ uint32_t quilt_band(const QuiltBinArgs& a, uint32_t g) {
  const uint32_t item = g / (uint32_t)a.H;
  return item * (uint32_t)a.bands_item + (g - item * (uint32_t)a.H) / (uint32_t)a.rows;
}

// Pass 1: entries per band (a workgroup histogram in LDS, one global add per
// band it touched).
__global__ void __launch_bounds__(256) k_qcount(QuiltBinArgs a) {
  extern __shared__ uint32_t qhist[];
  for (int k = threadIdx.x; k < a.bands; k += blockDim.x) qhist[k] = 0u;
  __syncthreads();
  const uint64_t npts = imin((int64_t)*a.n_points, a.cap);
  for (uint64_t c = (uint64_t)blockIdx.x * kQChunk; c < npts; c += (uint64_t)gridDim.x * kQChunk) {
    const uint64_t end = c + kQChunk < npts ? c + kQChunk : npts;
    for (uint64_t p = c + threadIdx.x; p < end; p += blockDim.x) {
      const uint2 pr = a.prows[p];
      if (pr.x != ~0u)
        for (uint32_t b = quilt_band(a, pr.x), b1 = quilt_band(a, pr.y); b <= b1; ++b) atomicAdd(&qhist[b], 1u);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < a.bands; k += blockDim.x)
    if (qhist[k]) atomicAdd(&a.band_cnt[k], qhist[k]);
}

// Pass 2 (one workgroup): band offsets and cursors, the overflow flag, and
// the bands sorted by decreasing entries (bitonic sort in LDS) so that the
// largest tiles start first.  Leaves the band counts at zero.
__global__ void __launch_bounds__(1024) k_qplan(QuiltBinArgs a) {
  constexpr int kPer = kQuiltBandCap / 1024;  // bands per thread
  __shared__ uint64_t sk[kQuiltBandCap];
  __shared__ uint64_t wtot[16];
  const int nb = a.bands, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  uint32_t c[kPer];
  uint64_t t = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int b = tid * kPer + k;
    c[k] = b < nb ? a.band_cnt[b] : 0u;
    t += c[k];
  }
  const uint64_t inc = wave_incl_scan(t);
  if (lane == 63) wtot[wv] = inc;
  __syncthreads();
  uint64_t run = inc - t, total = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wv) run += wtot[w];
    total += wtot[w];
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int b = tid * kPer + k;
    if (b < nb) {
      const uint32_t o = run < 0xFFFFFFFFull ? (uint32_t)run : 0xFFFFFFFFu;
      a.band_off[b] = o;
      a.band_cur[b] = o;
      a.band_cnt[b] = 0u;
      sk[b] = ((uint64_t)c[k] << 32) | (uint64_t)(0xFFFFFFFFu - (uint32_t)b);
    }
    run += c[k];
  }
  if (tid == 0) {
    const bool over = total > (uint64_t)a.entry_cap;
    a.band_off[nb] = over ? 0xFFFFFFFFu : (uint32_t)total;
    a.state[0] = over ? 1u : 0u;
    a.state[1] = total < 0xFFFFFFFFull ? (uint32_t)total : 0xFFFFFFFFu;
  }
  int n2 = 1;
  while (n2 < nb) n2 <<= 1;
  for (int b = nb + tid; b < n2; b += blockDim.x) sk[b] = 0ull;  // below every band's key
  __syncthreads();
  for (int size = 2; size <= n2; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int i = tid; i < n2; i += blockDim.x) {
        const int j = i ^ stride;
        if (j > i) {
          const uint64_t x = sk[i], y = sk[j];
          const bool desc = (i & size) == 0;
          if (desc ? x < y : x > y) {
            sk[i] = y;
            sk[j] = x;
          }
        }
      }
      __syncthreads();
    }
  for (int k = tid; k < nb; k += blockDim.x) a.order[k] = 0xFFFFFFFFu - (uint32_t)sk[k];
}

// Pass 3: the band lists.  A workgroup counts its points' entries per band in
// LDS, reserves each band's share with one global add, then places them.
__global__ void __launch_bounds__(256) k_qscatter(QuiltBinArgs a) {
  if (a.state[0]) return;  // overflow: the point splat takes the frame
  extern __shared__ uint32_t qsh[];
  uint32_t* hist = qsh;
  uint32_t* base = qsh + a.bands;
  for (int k = threadIdx.x; k < a.bands; k += blockDim.x) hist[k] = 0u;
  __syncthreads();
  const uint64_t npts = imin((int64_t)*a.n_points, a.cap);
  const uint64_t step = (uint64_t)gridDim.x * kQChunk;
  for (uint64_t c = (uint64_t)blockIdx.x * kQChunk; c < npts; c += step) {
    const uint64_t end = c + kQChunk < npts ? c + kQChunk : npts;
    for (uint64_t p = c + threadIdx.x; p < end; p += blockDim.x) {
      const uint2 pr = a.prows[p];
      if (pr.x != ~0u)
        for (uint32_t b = quilt_band(a, pr.x), b1 = quilt_band(a, pr.y); b <= b1; ++b) atomicAdd(&hist[b], 1u);
    }
  }
  __syncthreads();
  for (int k = threadIdx.x; k < a.bands; k += blockDim.x)
    if (hist[k]) {
      base[k] = atomicAdd(&a.band_cur[k], hist[k]);
      hist[k] = 0u;
    }
  __syncthreads();
  for (uint64_t c = (uint64_t)blockIdx.x * kQChunk; c < npts; c += step) {
    const uint64_t end = c + kQChunk < npts ? c + kQChunk : npts;
    for (uint64_t p = c + threadIdx.x; p < end; p += blockDim.x) {
      const uint2 pr = a.prows[p];
      if (pr.x != ~0u)
        for (uint32_t b = quilt_band(a, pr.x), b1 = quilt_band(a, pr.y); b <= b1; ++b)
          a.entries[base[b] + atomicAdd(&hist[b], 1u)] = (uint32_t)p;
    }
  }
}

// One tile per workgroup: clear the keys, splat the band's points into the
// tile's views and rows, write the tile out into its item's views.  kPBR:
// shaded colours.  Held to 128 VGPRs: four waves per SIMD.
template <bool kPBR, bool kHeld, int kBlock>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4))) k_splat_quilt(SplatArgs a) {
  extern __shared__ uint64_t qtile[];  // the tile's keys, then W column and H row ray slopes
  __shared__ uint32_t qnext;           // next unclaimed entry of the band
  if (*a.q_state != 0) return;         // overflow: the point splat takes the frame
  const Rig& trg = a.table_rig;
  const int32_t W = trg.W, H = trg.H;
  // Workgroups go to the 8 XCDs round robin (block b on XCD b % 8).  XCD x
  // takes the bands of rank x, x + 8, ... (ranks by decreasing size, so the
  // XCDs get equal shares), each band's view subsets on consecutive blocks of
  // that XCD: the subsets read the same points through one L2.  The grid is
  // padded to whole rounds of 8 bands; blocks past the last band exit.
  const uint32_t xcd = blockIdx.x & 7u, k = blockIdx.x >> 3;
  const uint32_t rank = (k / (uint32_t)a.q_subsets) * 8u + xcd, sub = k % (uint32_t)a.q_subsets;
  if (rank >= (uint32_t)a.q_bands) return;
  const int32_t band = (int32_t)a.q_order[rank];
  const int32_t item = band / a.q_bands_item, lband = band - item * a.q_bands_item;  // the band within its item
  QuiltTile qt;
  qt.keys = qtile;
  qt.rows = a.q_rows;
  qt.y_lo = lband * a.q_rows;
  qt.y_hi = min(H - 1, qt.y_lo + a.q_rows - 1);
  qt.r_lo = (int32_t)sub * a.q_views;
  qt.r_hi = min(trg.n_views, qt.r_lo + a.q_views);
  const int32_t nkeys = a.q_rows * a.q_views * W;
  float* tx = reinterpret_cast<float*>(qtile + nkeys);
  float* ty = tx + W;
  for (int32_t k = threadIdx.x; k < nkeys; k += blockDim.x) qtile[k] = ~0ull;
  for (int k = threadIdx.x; k < W; k += blockDim.x) tx[k] = ((float)k + 0.5f - trg.cx) / trg.fx;
  for (int k = threadIdx.x; k < H; k += blockDim.x) ty[k] = ((float)k + 0.5f - trg.cy) / trg.fy;
  if (threadIdx.x == 0) qnext = 0u;
  __syncthreads();
  const uint32_t e0 = a.q_band_off[band], e1 = a.q_band_off[band + 1];
  const Item it0 = load_uniform(a.items + item);
  const int lane = threadIdx.x & 63;
  uint32_t written = 0;
  uint32_t* const queue = kHeld ? nullptr : reinterpret_cast<uint32_t*>(ty + H) + (threadIdx.x >> 6) * kSplatQueue;
  // the band's entries in chunks of 64, one chunk per wave at a time, taken
  // from an LDS counter as the waves free up: the tile ends when its last
  // chunk does, whatever the per-point work
  for (;;) {
    uint32_t c = 0;
    if (lane == 0) c = atomicAdd(&qnext, 64u);
    c = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
    if (c >= e1 - e0) break;
    const uint32_t e = e0 + c + (uint32_t)lane;
    const bool valid = e < e1;
    const uint32_t p = a.q_entries[valid ? e : e1 - 1];
    const Point pt = a.points[p];
    const TriRec T = a.rec[pt.tri_flags & 0x0FFFFFFFu];
    qt.box = a.pbox + p;
    splat_wave<kPBR, true, kHeld>(it0, valid, p, pt, T, tx, ty, a, queue, nullptr, qt.r_lo, qt.r_hi, written, &qt);
  }
  __syncthreads();
  // the tile as RGBA8 (+ depth): one pixel row of one view per wave at a time
  const int32_t nrows = qt.y_hi - qt.y_lo + 1, nvt = qt.r_hi - qt.r_lo;
  const int wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int32_t q = wv; q < nvt * nrows; q += nw) {
    const int32_t rv = q / nrows, yy = q - rv * nrows;
    const uint64_t* src = qtile + (rv * a.q_rows + yy) * W;
    const int64_t o = (((int64_t)item * trg.n_views + qt.r_lo + rv) * H + (qt.y_lo + yy)) * W;
    for (int32_t x = lane; x < W; x += 64) {
      const uint64_t key = src[x];
      const bool empty = key == ~0ull;
      a.out_rgba[o + x] = empty ? 0u : (uint32_t)key;
      if (a.out_depth) a.out_depth[o + x] = empty ? __uint_as_float(0x7f800000u) : __uint_as_float((uint32_t)(key >> 32));
    }
  }
  if (lane == 0) line_add(a.stats, LINE_WRITTEN, written);
}

// ------------------------------------------------------------------ a3: splat, triangle-major
//
// The same splats and keys as k_splat, visited per (triangle, view) instead of
// per point.  A wave takes 64 (triangle, view) pairs; each lane sets its pair
// up (visibility, Q8 vertices, edge functions, pixel bounding box) and the
// wave then walks the concatenated bounding boxes 64 pixels at a time, so that
// every lane works whatever the boxes' sizes.  A pixel inside the triangle
// finds its owning cell by the clamped lattice coordinates of its ray hit
// (row table of the triangle), then applies that point's splat rectangle and
// colour (Eqs. 8-9) from the point's PointBox, and the 64-bit depth test.

// Everything the pixel pass needs of one (triangle, view) pair, in LDS.
struct alignas(16) PairData {
  int32_t qx0, qx1, qx2, qy0;    // Q8 vertices, positively oriented
  int32_t qy1, qy2, xy0, w;      // bounding box origin (x | y << 16) and width
  float delta, cu, cw, ks;       // plane distance of the eye, lattice offsets, lens shift
  float fxfy_ad, b, inv_w, acell;  // fx*fy*|delta| (Eq. 8), eye offset, 1/width, 1/(Sx*Sy)
  uint64_t* kv;                  // keys of this view
  int32_t row_stride;            // keys per pixel row
  float suv;                     // acell * ruv (Eq. 8)
  float nx, ny, nz, ux;          // the triangle's plane and lattice axes
  float uy, uz, wx, wy;
  float wz, sx, sy, ruv;
  float smin, smax, irange;      // Eqs. 4-5, 9
  int32_t jlo;                   // first lattice row
  uint64_t first;                // the triangle's first point
  int32_t jhi, pad;
};
static_assert(sizeof(PairData) == 160, "PairData is ten 16-byte words");
constexpr int kPairWords = 10;

// The pair records of a wave are kept in LDS word-major: word g of pair o at
// [g][o], so that lanes reading consecutive pairs hit consecutive banks.
__device__ __forceinline__ void store_pair(uint4 (*pw)[64], int o, const PairData& P) {
  const uint4* w = reinterpret_cast<const uint4*>(&P);
#pragma unroll
  for (int g = 0; g < kPairWords; ++g) pw[g][o] = w[g];
}

__device__ __forceinline__ PairData load_pair(const uint4 (*pw)[64], int o) {
  PairData P;
  uint4* w = reinterpret_cast<uint4*>(&P);
#pragma unroll
  for (int g = 0; g < kPairWords; ++g) w[g] = pw[g][o];
  return P;
}

// One covered pixel of pair Q: ray hit, owning cell, its splat rectangle and
// colour (Eqs. 8-9), the 64-bit depth test.  Returns 1 when a key was written.
__device__ __forceinline__ uint32_t splat_fragment(const PairData& Q, int32_t x, int32_t y, const float* tx,
                                                   const float* ty, const RowEntry* __restrict__ rows,
                                                   const PointBox* __restrict__ pbox) {
  const float rx = tx[x] - Q.ks, ry = ty[y];
  const float den = (Q.nx * rx + Q.ny * ry) + Q.nz;
  const float Z = Q.delta / den;
  if (!(Z > 0.0f) || isinf(Z)) return 0;
  const float ur = (Q.ux * rx + Q.uy * ry) + Q.uz;
  const float wr = (Q.wx * rx + Q.wy * ry) + Q.wz;
  const float sv = Q.sx * (Z * ur + Q.cu) + 0.5f;
  const float tv = Q.sy * (Z * wr + Q.cw) + 0.5f;
  // owning cell: clamp to the lattice rows, then to the row's cells
  int32_t cj = (int32_t)floorf(clamp_big(tv));
  cj = cj < Q.jlo ? Q.jlo : (cj > Q.jhi ? Q.jhi : cj);
  const RowEntry R = rows[Q.first + (uint64_t)(cj - Q.jlo)];
  int32_t ci = (int32_t)floorf(clamp_big(sv));
  ci = ci < R.ilo ? R.ilo : (ci > R.ihi ? R.ihi : ci);
  const PointBox& B = pbox[Q.first + R.start + (uint32_t)(ci - R.ilo)];
  const int32_t rws = B.rows;
  if (rws != kAllRows) {
    const int32_t r0 = (int16_t)(rws & 0xFFFF), r1 = (int16_t)((uint32_t)rws >> 16);
    if (y < r0 || y > r1) return 0;
    const float b = Q.b;
    float xmn = B.cA[0] - b * B.cC[0], xmx = xmn;
#pragma unroll
    for (int kk = 1; kk < 4; ++kk) {
      const float xx = B.cA[kk] - b * B.cC[kk];
      xmn = xx < xmn ? xx : xmn;
      xmx = xx > xmx ? xx : xmx;
    }
    if (x < (int32_t)ceilf(clamp_big(xmn - 0.515625f)) || x > (int32_t)floorf(clamp_big(xmx - 0.484375f))) return 0;
  }
  // colour of the point in this view (Eqs. 8-9)
  const float Ar = B.zc3 / Q.fxfy_ad;
  const float vse = Q.acell < Ar ? Q.ruv * Ar : Q.suv;
  const float vs = vse < Q.smin ? Q.smin : (vse > Q.smax ? Q.smax : vse);
  const float tau = (vs - Q.smin) * Q.irange;
  int32_t tq = (int32_t)floorf(tau * 256.0f + 0.5f);
  tq = tq < 0 ? 0 : (tq > 256 ? 256 : tq);
  const uint32_t wa = (uint32_t)(256 - tq), wz = (uint32_t)tq;
  const uint32_t lo = B.tvmin, hi = B.tvmax;
  const uint32_t col =
      ((((lo & 0x00FF00FFu) * wa + (hi & 0x00FF00FFu) * wz + 0x00800080u) >> 8) & 0x00FF00FFu) |
      (((((lo >> 8) & 0x00FF00FFu) * wa + ((hi >> 8) & 0x00FF00FFu) * wz + 0x00800080u) >> 8) & 0x00FF00FFu) << 8;
  key_min(&Q.kv[(int64_t)y * Q.row_stride + x], ((uint64_t)__float_as_uint(Z) << 32) | col);
  return 1;
}

template <bool kMulti>
__global__ void __launch_bounds__(256) k_splat_tv(SplatArgs a) {
  extern __shared__ float ray_tab[];  // W column slopes, then H row slopes
  __shared__ uint4 pd[4][kPairWords][64];
  __shared__ uint32_t poff[4][64];
  __shared__ uint32_t fq[4][128];     // covered pixels waiting: pair | x << 6 | y << 19
  const Rig& trg = a.table_rig;
  float* tx = ray_tab;
  float* ty = ray_tab + trg.W;
  for (int k = threadIdx.x; k < trg.W; k += blockDim.x) tx[k] = ((float)k + 0.5f - trg.cx) / trg.fx;
  for (int k = threadIdx.x; k < trg.H; k += blockDim.x) ty[k] = ((float)k + 0.5f - trg.cy) / trg.fy;
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  const int32_t V = trg.n_views;
  const int64_t npairs = (int64_t)imin((int64_t)*a.n_tris, a.nt) * V;
  const Item it0 = load_uniform(a.items);
  uint4 (*const mypd)[64] = pd[wv];
  uint32_t* const myoff = poff[wv];
  uint32_t* const myq = fq[wv];
  uint32_t written = 0, covered = 0;  // key updates; covered pixels visited (the hole census)
  const int64_t chunks = (npairs + 63) >> 6;
  for (int64_t c = (int64_t)blockIdx.x * 4 + wv; c < chunks; c += (int64_t)gridDim.x * 4) {
    // ---- phase A: one (triangle, view) pair per lane
    const int64_t k = c * 64 + lane;
    uint32_t npx = 0;
    PairData P;
    if (k < npairs) {
      const uint32_t ti = (uint32_t)k / (uint32_t)V;
      const int32_t r = (int32_t)((uint32_t)k - ti * (uint32_t)V);
      const uint32_t tri = a.tris[ti];
      const TriRec& T = a.rec[tri];
      const Item& it = kMulti ? a.items[T.item] : it0;
      const Rig& rg = it.rig;
      // every point of the triangle must be in the buffer (else the frame
      // overflowed and the triangle is left out)
      const uint64_t first = a.offsets[tri];
      const bool fits = first + a.counts[tri] <= (uint64_t)a.cap;
      const float b = fits && r < rg.n_views ? rg.eye[r] : 0.0f;
      const float delta = T.h - T.nx * b;
      const int32_t H8 = 256 * rg.H, W8 = 256 * rg.W;
      bool act = fits && r < rg.n_views && faces_eye(T.p0x, T.p0y * T.p0y, T.p0z * T.p0z, delta, b);
      int32_t qx[3], qy[3];
      if (act) act = q8_xy(T.a0, T.c0, T.y0, b, qx[0], qy[0]) && q8_xy(T.a1, T.c1, T.y1, b, qx[1], qy[1]) &&
                     q8_xy(T.a2, T.c2, T.y2, b, qx[2], qy[2]);
      if (act && ((qx[0] < 0 && qx[1] < 0 && qx[2] < 0) || (qx[0] > W8 && qx[1] > W8 && qx[2] > W8) ||
                  (qy[0] < 0 && qy[1] < 0 && qy[2] < 0) || (qy[0] > H8 && qy[1] > H8 && qy[2] > H8)))
        act = false;
      if (act) {
        const int64_t a2 = (int64_t)(qx[1] - qx[0]) * (qy[2] - qy[0]) - (int64_t)(qy[1] - qy[0]) * (qx[2] - qx[0]);
        if (a2 == 0) act = false;
        if (a2 < 0) {
          int32_t u = qx[1]; qx[1] = qx[2]; qx[2] = u;
          u = qy[1]; qy[1] = qy[2]; qy[2] = u;
        }
      }
      if (act) {
        const int32_t xmin = min(qx[0], min(qx[1], qx[2])), xmax = max(qx[0], max(qx[1], qx[2]));
        const int32_t ymin = min(qy[0], min(qy[1], qy[2])), ymax = max(qy[0], max(qy[1], qy[2]));
        const int32_t X0 = max(0, -((128 - xmin) >> 8)), X1 = min(rg.W - 1, (xmax - 128) >> 8);
        const int32_t Y0 = max(0, -((128 - ymin) >> 8)), Y1 = min(rg.H - 1, (ymax - 128) >> 8);
        if (X0 <= X1 && Y0 <= Y1) {
          const int32_t w = X1 - X0 + 1;
          npx = (uint32_t)(w * (Y1 - Y0 + 1));
          P.qx0 = qx[0]; P.qx1 = qx[1]; P.qx2 = qx[2];
          P.qy0 = qy[0]; P.qy1 = qy[1]; P.qy2 = qy[2];
          P.xy0 = X0 | (Y0 << 16);
          P.w = w;
          P.delta = delta;
          P.cu = T.ux * (b - T.p0x) - T.cu0;
          P.cw = T.wx * (b - T.p0x) - T.cw0;
          P.ks = rg.kshift[r];
          P.fxfy_ad = rg.fxfy * fabsf(delta);
          P.b = b;
          P.inv_w = 1.0f / (float)w;
          const bool rowmajor = it.key_layout != 0;
          P.kv = it.keys + (rowmajor ? (int64_t)r * rg.W : (int64_t)r * rg.W * rg.H);
          P.row_stride = rowmajor ? rg.n_views * rg.W : rg.W;
          P.acell = 1.0f / (T.sx * T.sy);
          P.suv = P.acell * T.ruv;
          P.nx = T.nx; P.ny = T.ny; P.nz = T.nz;
          P.ux = T.ux; P.uy = T.uy; P.uz = T.uz;
          P.wx = T.wx; P.wy = T.wy; P.wz = T.wz;
          P.sx = T.sx; P.sy = T.sy; P.ruv = T.ruv;
          P.smin = T.smin; P.smax = T.smax; P.irange = T.irange;
          const int2 jr = *reinterpret_cast<const int2*>(&a.em[tri].jlo);
          P.jlo = jr.x;
          P.jhi = jr.y;
          P.first = first;
          P.pad = 0;
        }
      }
    }
    // exclusive offsets of the pixel boxes; pair data to LDS
    uint32_t inc = npx;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(inc, d, 64);
      if (lane >= d) inc += o;
    }
    const uint32_t total = __shfl(inc, 63, 64);
    if (total == 0) continue;
    myoff[lane] = inc - npx;
    if (npx) store_pair(mypd, lane, P);
    wave_sync_lds();
    // ---- phase B: 64 box pixels per round over the concatenated boxes; the
    // covered ones queue up and are splatted 64 at a time
    uint32_t qn = 0;
    for (uint32_t base = 0; base < total; base += 64) {
      const uint32_t u = base + lane;
      bool cov = false;
      uint32_t entry = 0;
      if (u < total) {
        int o = 0;
#pragma unroll
        for (int st = 32; st >= 1; st >>= 1)
          if (myoff[o + st] <= u) o += st;
        const uint4 g0 = mypd[0][o], g1 = mypd[1][o];
        const float inv_w = __uint_as_float(mypd[3][o].z);
        const int32_t q = (int32_t)(u - myoff[o]);
        const int32_t w = (int32_t)g1.w, xy0 = (int32_t)g1.z;
        int32_t yq = (int32_t)((float)q * inv_w);
        int32_t xq = q - yq * w;
        if (xq < 0) { yq -= 1; xq += w; }
        else if (xq >= w) { yq += 1; xq -= w; }
        const int32_t x = (xy0 & 0xFFFF) + xq, y = (xy0 >> 16) + yq;
        const int32_t pxq = 256 * x + 128, pyq = 256 * y + 128;
        const int32_t qx0 = (int32_t)g0.x, qx1 = (int32_t)g0.y, qx2 = (int32_t)g0.z, qy0 = (int32_t)g0.w,
                      qy1 = (int32_t)g1.x, qy2 = (int32_t)g1.y;
        // edge functions in 64-bit integers; an edge owns its ties iff dy > 0 || (dy == 0 && dx > 0)
        auto inside = [](int32_t ax, int32_t ay, int32_t bx, int32_t by, int32_t px, int32_t py) {
          const int32_t dx = bx - ax, dy = by - ay;
          const int64_t E = (int64_t)dx * (py - ay) - (int64_t)dy * (px - ax);
          return E > 0 || (E == 0 && (dy > 0 || (dy == 0 && dx > 0)));
        };
        cov = inside(qx0, qy0, qx1, qy1, pxq, pyq) && inside(qx1, qy1, qx2, qy2, pxq, pyq) &&
              inside(qx2, qy2, qx0, qy0, pxq, pyq);
        entry = (uint32_t)o | ((uint32_t)x << 6) | ((uint32_t)y << 19);
      }
      const uint64_t m = __builtin_amdgcn_ballot_w64(cov);
      if (cov) myq[qn + (uint32_t)__builtin_popcountll(m & below)] = entry;
      qn += (uint32_t)__builtin_popcountll(m);
      if (qn >= 64) {
        wave_sync_lds();
        const uint32_t e = myq[lane];
        covered += 1;
        written += splat_fragment(load_pair(mypd, (int)(e & 63)), (int32_t)((e >> 6) & 0x1FFF), (int32_t)(e >> 19), tx,
                                  ty, a.rows, a.pbox);
        const uint32_t rest = qn - 64;
        const uint32_t moved = lane < rest ? myq[64 + lane] : 0u;
        wave_sync_lds();
        if (lane < rest) myq[lane] = moved;
        qn = rest;
      }
    }
    if (qn) {
      wave_sync_lds();
      if ((uint32_t)lane < qn) {
        const uint32_t e = myq[lane];
        covered += 1;
        written += splat_fragment(load_pair(mypd, (int)(e & 63)), (int32_t)((e >> 6) & 0x1FFF), (int32_t)(e >> 19), tx,
                                  ty, a.rows, a.pbox);
      }
    }
    wave_sync_lds();  // the pair data and the queue are rewritten for the next chunk
  }
  const uint64_t wsum = wave_sum((uint64_t)written), csum = wave_sum((uint64_t)covered);
  if (lane == 0) line_add(a.stats, LINE_WRITTEN, wsum);
  if (lane == 0) line_add(a.stats, LINE_COVERED, csum);
}

// keys -> RGBA8 (+ depth) in [item][view][y][x] order; keys re-cleared.
__global__ void k_resolve(uint64_t* __restrict__ keys, int64_t n, int32_t nv, int32_t H, int32_t W, int32_t layout,
                          uint32_t* __restrict__ rgba, float* __restrict__ depth, const uint32_t* __restrict__ gate) {
  if (gate && *gate == 0) return;
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t per_view = (int64_t)W * H, per_item = per_view * nv;
  for (; i < n; i += stride) {
    int64_t k = i;
    if (layout) {
      const int64_t b = i / per_item, rem = i % per_item;
      const int64_t r = rem / per_view, q = rem % per_view;
      const int64_t y = q / W, x = q % W;
      k = b * per_item + (y * nv + r) * W + x;
    }
    const uint64_t key = keys[k];
    const bool empty = key == ~0ull;
    rgba[i] = empty ? 0u : (uint32_t)key;
    if (depth) depth[i] = empty ? __uint_as_float(0x7f800000u) : __uint_as_float((uint32_t)(key >> 32));
    keys[k] = ~0ull;
  }
}

// ------------------------------------------------------------------ a4: interleave + reconstruction

// Logical block of a 1-D launch of nb blocks such that the blocks the
// hardware places on one XCD (round robin over 8) take one contiguous eighth
// of the logical order: neighbouring tiles share that XCD's L2.
__device__ __forceinline__ uint32_t xcd_block(uint32_t b, uint32_t nb) {
  const uint32_t per = nb / 8, extra = nb % 8, xcd = b % 8, k = b / 8;
  // XCD x takes per (+1 for the first `extra`) consecutive logical blocks
  return xcd * per + (xcd < extra ? xcd : extra) + k;
}

// floor(a / b) for 0 <= a < 2^52 with a quotient below 2^31, b > 0, rb = 1.0 / b:
// the product is within one of the floor, and the remainder's low 32 bits settle it.
__device__ __forceinline__ int32_t quotient_by(int64_t a, int32_t b, double rb) {
  int32_t q = (int32_t)((double)a * rb);
  const int32_t r = (int32_t)((uint32_t)a - (uint32_t)q * (uint32_t)b);
  return r < 0 ? q - 1 : (r >= b ? q + 1 : q);
}

// x clamped to [0, hi], hi >= 0
__device__ __forceinline__ int32_t clamp0(int32_t x, int32_t hi) {
  int32_t d;
  asm("v_med3_i32 %0, %1, 0, %2" : "=v"(d) : "v"(x), "v"(hi));
  return d;
}

// Four panel pixels' twelve bytes to row Y, column X0 (nx of them inside the
// panel): three 32-bit words where they are aligned and whole.
__device__ __forceinline__ void store_panel(const InterleaveArgs& a, int64_t Y, int64_t X0, int nx, const uint32_t bytes[12]) {
  uint8_t* dst = a.panel + (Y * a.Wp + X0) * 3;
  if (nx == 4 && ((uintptr_t)dst & 3) == 0) {
    uint32_t* d32 = reinterpret_cast<uint32_t*>(dst);
    d32[0] = bytes[0] | (bytes[1] << 8) | (bytes[2] << 16) | (bytes[3] << 24);
    d32[1] = bytes[4] | (bytes[5] << 8) | (bytes[6] << 16) | (bytes[7] << 24);
    d32[2] = bytes[8] | (bytes[9] << 8) | (bytes[10] << 16) | (bytes[11] << 24);
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k)
      if (k < 3 * nx) dst[k] = (uint8_t)bytes[k];
  }
}

// One lane per four consecutive panel pixels.  Panel rows are spread over the
// XCDs in contiguous bands so that each view row is fetched into one L2.
// View stacks of less than 4 GiB whose planes are below 16 MiB (the rule is
// launch_interleave's): a tap's byte is loaded from a 32-bit offset, view * plane + (row +
// column) with the row the same for the whole workgroup and the column for a
// pixel's three channels, so a tap costs five vector instructions instead of
// some 25 of 64-bit address arithmetic, which bounded the eight-tap modes
// (panel of 2560 x 1600 from 48 views of 512 x 512: 95 -> 51 us; one tap: 23 ->
// 18 us).
template <int kTaps>
__global__ void __launch_bounds__(256) k_interleave_small(InterleaveArgs a, uint32_t blocks_per_row, uint32_t nblocks) {
  const uint32_t L = xcd_block(blockIdx.x, nblocks);
  const int32_t Y = (int32_t)(L / blocks_per_row);
  const int32_t X0 = (int32_t)(((L % blocks_per_row) * blockDim.x + threadIdx.x) * 4);
  const int32_t yq = __builtin_amdgcn_readfirstlane(quotient_by((2 * Y + 1) * (int64_t)a.Hv * 128, a.Hp, 1.0 / (double)a.Hp));
  uint32_t row[kTaps];  // byte offset of each tap's view row
#pragma unroll
  for (int t = 0; t < kTaps; ++t)
    row[t] = (uint32_t)(4 * a.Wv * max(0, min(a.Hv - 1, (yq + (kTaps > 1 ? a.dy[t] : 0)) >> 8)));
  if (X0 >= a.Wp) return;
  const int nx = min(4, a.Wp - X0);
  const uint32_t plane = 4u * (uint32_t)a.Wv * (uint32_t)a.Hv;
  const double rwp = 1.0 / (double)a.Wp;
  const int32_t v_last = a.V - 1, x_last = a.Wv - 1;
  const uint8_t* const src = reinterpret_cast<const uint8_t*>(a.views);
  uint32_t bytes[12];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int32_t X = min(X0 + k, a.Wp - 1);  // a pixel beyond the panel repeats the last one
    const int32_t xq = quotient_by((2 * X + 1) * (int64_t)a.Wv * 128, a.Wp, rwp);
    uint32_t at[kTaps];
#pragma unroll
    for (int t = 0; t < kTaps; ++t)
      at[t] = row[t] + 4u * (uint32_t)clamp0((xq + (kTaps > 1 ? a.dx[t] : 0)) >> 8, x_last);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint32_t phi = (uint32_t)(3 * X + c) * a.K1 + (uint32_t)Y * a.Ky + a.K0;
      const uint32_t uh = __umulhi(phi, (uint32_t)a.V), ul = phi * (uint32_t)a.V;
      uint32_t sum = 0;
#pragma unroll
      for (int t = 0; t < kTaps; ++t) {
        int32_t v = (int32_t)uh;
        if (kTaps > 1) {
          const uint32_t dl = (uint32_t)a.du[t];
          v += (int32_t)(a.du[t] >> 32) + (ul + dl < dl ? 1 : 0);
          v = clamp0(v, v_last);
        }
        sum += src[__umul24((uint32_t)v, plane) + at[t] + (uint32_t)c];
      }
      bytes[3 * k + c] = kTaps > 1 ? (sum + 4u) >> 3 : sum;
    }
  }
  store_panel(a, Y, X0, nx, bytes);
}

// Larger stacks: 64-bit addresses.
__global__ void __launch_bounds__(256) k_interleave(InterleaveArgs a, uint32_t blocks_per_row, uint32_t nblocks) {
  const uint32_t L = xcd_block(blockIdx.x, nblocks);
  const int64_t Y = L / blocks_per_row;
  const int64_t X0 = ((int64_t)(L % blocks_per_row) * blockDim.x + threadIdx.x) * 4;
  if (Y >= a.Hp || X0 >= a.Wp) return;
  const int64_t yq = ((2 * Y + 1) * (int64_t)a.Hv * 128) / a.Hp;
  uint32_t bytes[12];
  const int nx = a.Wp - X0 < 4 ? (int)(a.Wp - X0) : 4;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int64_t X = X0 + k;
    const int64_t xq = ((2 * X + 1) * (int64_t)a.Wv * 128) / a.Wp;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      uint32_t val = 0;
      if (k < nx) {
        const uint32_t phi = (uint32_t)(3 * X + c) * a.K1 + (uint32_t)Y * a.Ky + a.K0;
        const uint64_t U = (uint64_t)phi * (uint64_t)a.V;
        if (a.mode == 0) {
          const int64_t v = (int64_t)(U >> 32);
          val = (a.views[(v * a.Hv + (yq >> 8)) * a.Wv + (xq >> 8)] >> (8 * c)) & 255u;
        } else {
          uint32_t sum = 0;
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            int64_t v = ((int64_t)U + a.du[t]) >> 32;
            int64_t x = (xq + a.dx[t]) >> 8, y = (yq + a.dy[t]) >> 8;
            v = v < 0 ? 0 : (v > a.V - 1 ? a.V - 1 : v);
            x = x < 0 ? 0 : (x > a.Wv - 1 ? a.Wv - 1 : x);
            y = y < 0 ? 0 : (y > a.Hv - 1 ? a.Hv - 1 : y);
            sum += (a.views[(v * a.Hv + y) * a.Wv + x] >> (8 * c)) & 255u;
          }
          val = (sum + 4u) >> 3;
        }
      }
      bytes[3 * k + c] = val;
    }
  }
  store_panel(a, Y, X0, nx, bytes);
}

// Angular supersampling filter, one lane per four consecutive pixels of an
// output view (16-byte loads and stores where whole).  Per channel the
// weighted sum fits 32 bits (weights < 2^16, at most 3S sub-views); the
// rounded quotient (acc + ws/2) div ws is taken exactly from a double
// reciprocal and one integer correction step.
__global__ void __launch_bounds__(256) k_angular_filter(AngularArgs a) {
  const int v = blockIdx.y;
  const int64_t npx = (int64_t)a.W * a.H;
  const int64_t p0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  if (p0 >= npx) return;
  const int n = a.cnt[v];
  uint32_t ws = 0;
  for (int e = 0; e < n; ++e) ws += a.wt[v * a.maxe + e];
  const double rcp = 1.0 / (double)ws;
  const uint32_t half = ws / 2;
  const bool whole = p0 + 4 <= npx && (npx & 3) == 0;
  uint32_t acc[4][4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[k][c] = 0u;
  for (int e = 0; e < n; ++e) {
    const uint32_t w = a.wt[v * a.maxe + e];
    const uint32_t* row = a.sub + (int64_t)a.src[v * a.maxe + e] * npx + p0;
    uint32_t px[4];
    if (whole) {
      const uint4 q = *reinterpret_cast<const uint4*>(row);
      px[0] = q.x; px[1] = q.y; px[2] = q.z; px[3] = q.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) px[k] = p0 + k < npx ? row[k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[k][c] += w * ((px[k] >> (8 * c)) & 255u);
  }
  uint32_t o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    o[k] = 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t num = acc[k][c] + half;
      uint32_t q = (uint32_t)((double)num * rcp);
      const int64_t r = (int64_t)num - (int64_t)q * ws;
      if (r >= (int64_t)ws) q += 1;
      else if (r < 0) q -= 1;
      o[k] |= q << (8 * c);
    }
  }
  uint32_t* dst = a.out + (int64_t)v * npx + p0;
  if (whole) {
    *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
  } else {
    for (int k = 0; k < 4; ++k)
      if (p0 + k < npx) dst[k] = o[k];
  }
}

// ------------------------------------------------------------------ launchers

static inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

void launch_fill_u64(uint64_t* p, int64_t n, uint64_t v, hipStream_t s) {
  if (n <= 0) return;
  unsigned g = (unsigned)imin(nblk(n, 256), 256 * 64);
  k_fill_u64<<<g, 256, 0, s>>>(p, n, v);
}

void launch_store_item(const Item& it, Item* dst, hipStream_t s) { k_store_item<<<1, 64, 0, s>>>(it, dst); }

void launch_export_stats(const uint64_t* st, int64_t cap, int64_t* out, hipStream_t s) {
  k_export_stats<<<1, 64, 0, s>>>(st, cap, out);
}

void launch_build_mip(const uint32_t* src, uint32_t* dst, int s, hipStream_t st) {
  int64_t n = (int64_t)(s >> 1) * (s >> 1);
  k_build_mip<<<nblk(n, 256), 256, 0, st>>>(src, dst, s);
}

// Below kSplitTris triangles (two waves per SIMD at one lane each) eight lanes
// share a triangle's views.
constexpr int64_t kSplitTris = 131072;

int setup_lanes(int64_t nt) { return nt < kSplitTris ? 8 : 1; }

// Set-up workgroups whose sums the last of them scans.
constexpr unsigned kScanTiles = 256;
static bool setup_scans(int64_t nt) { return nt > 0 && setup_lanes(nt) == 8 && nblk(nt, 256 / 8) <= kScanTiles; }

void launch_tri_setup(const SetupArgs& args, hipStream_t s) {
  if (args.nt <= 0) return;
  SetupArgs a = args;
  a.ticket = setup_scans(a.nt) ? reinterpret_cast<uint32_t*>(a.stats + STAT_TICKET) : nullptr;
  const int vl = setup_lanes(a.nt);
  const unsigned g = nblk(a.nt, 256 / vl);
  if (a.n_items > 1 && vl == 8)
    k_tri_setup<true, 8><<<g, 256, 0, s>>>(a);
  else if (a.n_items > 1)
    k_tri_setup<true, 1><<<g, 256, 0, s>>>(a);
  else if (vl == 8)
    k_tri_setup<false, 8><<<g, 256, 0, s>>>(a);
  else
    k_tri_setup<false, 1><<<g, 256, 0, s>>>(a);
}

void launch_interleave_batch(const InterleaveArgs& a, int n_items, int64_t view_stride, int64_t panel_stride,
                             hipStream_t s) {
  for (int b = 0; b < n_items; ++b) {
    InterleaveArgs c = a;
    c.views = a.views + view_stride * b;
    c.panel = a.panel + panel_stride * b;
    launch_interleave(c, s);
  }
}

void launch_scan(uint64_t* tile_sum, const uint64_t* tile_stat, int64_t nt, uint64_t* stats, hipStream_t s) {
  const int64_t per = 256 / setup_lanes(nt);
  if (setup_scans(nt)) return;
  k_scan_top<<<1, 1024, 0, s>>>(tile_sum, tile_stat, (nt + per - 1) / per, stats);
}

void launch_emit(const EmitArgs& a, int fetch_blocks, hipStream_t s) {
  if (a.nt <= 0) return;
  // the set-up's tiles: 32 triangles spread the rows of a small scene over more workgroups
  const int tile = 256 / setup_lanes(a.nt);
  const unsigned g = kEmitBigBlocks + nblk(a.nt, tile);
  if (tile == 32) k_emit<32><<<g, 256, 0, s>>>(a);
  else k_emit<256><<<g, 256, 0, s>>>(a);
  if (a.pbox && a.tm)
    k_fetch<true, true><<<fetch_blocks, 256, 0, s>>>(a);
  else if (a.pbox)
    k_fetch<true, false><<<fetch_blocks, 256, 0, s>>>(a);
  else if (a.tm)
    k_fetch<false, true><<<fetch_blocks, 256, 0, s>>>(a);
  else
    k_fetch<false, false><<<fetch_blocks, 256, 0, s>>>(a);
}

// Four workgroups of the point splat fit a CU; more would find their queues empty.
constexpr int kSplatGrid = 1024;

void launch_splat(const SplatArgs& a, int grid_blocks, hipStream_t s) {
  size_t lds = sizeof(float) * (size_t)(a.table_rig.W + a.table_rig.H);
  if (a.pbox && !a.tm) {
    if (a.n_items > 1)
      k_splat_tv<true><<<grid_blocks, 256, lds, s>>>(a);
    else
      k_splat_tv<false><<<grid_blocks, 256, lds, s>>>(a);
    return;
  }
  grid_blocks = grid_blocks < kSplatGrid ? grid_blocks : kSplatGrid;
  if (a.n_items > 1 && a.tm)
    k_splat<true, true><<<grid_blocks, 256, lds, s>>>(a);
  else if (a.n_items > 1)
    k_splat<true, false><<<grid_blocks, 256, lds, s>>>(a);
  else if (a.tm)
    k_splat<false, true><<<grid_blocks, 256, lds, s>>>(a);
  else
    k_splat<false, false><<<grid_blocks, 256, lds, s>>>(a);
}

void launch_resolve(uint64_t* keys, int64_t n_items, int32_t n_views, int32_t H, int32_t W, int32_t key_layout,
                    uint32_t* rgba, float* depth, hipStream_t s, const uint32_t* gate) {
  const int64_t n = n_items * n_views * (int64_t)H * W;
  // a gated resolve is a fallback that nearly always exits at once: a small grid
  unsigned g = (unsigned)imin(nblk(n, 256), gate ? 1024 : 256 * 64);
  k_resolve<<<g, 256, 0, s>>>(keys, n, n_views, H, W, key_layout, rgba, depth, gate);
}

constexpr size_t kQuiltStaticLds = 16;  // the workgroup's entry counter

size_t quilt_lds_bytes(int32_t rows, int32_t views, int32_t W, int32_t H) {
  return (size_t)rows * (size_t)views * (size_t)W * 8u + (size_t)(W + H) * 4u + kQuiltStaticLds;
}

size_t quilt_queue_bytes(int32_t block) { return (size_t)(block / 64) * kSplatQueue * sizeof(uint32_t); }

void launch_quilt_bin(const QuiltBinArgs& a, hipStream_t s) {
  const unsigned g = (unsigned)imin(nblk(a.cap, kQChunk), 1024);
  k_qcount<<<g, 256, sizeof(uint32_t) * (size_t)a.bands, s>>>(a);
  k_qplan<<<1, 1024, 0, s>>>(a);
  k_qscatter<<<g, 256, 2 * sizeof(uint32_t) * (size_t)a.bands, s>>>(a);
}

// The tile kernel of a frame: shaded or not, the queues of covered pixels in
// LDS or (1024 threads only) held in registers.
using QuiltKernel = void (*)(SplatArgs);
static QuiltKernel quilt_kernel(bool pbr, bool queue, int block) {
  if (block == 512) return pbr ? k_splat_quilt<true, false, 512> : k_splat_quilt<false, false, 512>;
  if (queue) return pbr ? k_splat_quilt<true, false, 1024> : k_splat_quilt<false, false, 1024>;
  return pbr ? k_splat_quilt<true, true, 1024> : k_splat_quilt<false, true, 1024>;
}

hipError_t prepare_quilt_kernels(size_t lds) {
  const int dyn = (int)(lds - kQuiltStaticLds);
  for (int k = 0; k < 6; ++k) {
    const QuiltKernel f = quilt_kernel(k & 1, k < 4, k < 2 ? 512 : 1024);
    const hipError_t e = hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_splat_quilt(const SplatArgs& a, hipStream_t s) {
  const size_t lds = quilt_lds_bytes(a.q_rows, a.q_views, a.table_rig.W, a.table_rig.H) - kQuiltStaticLds +
                     (a.q_queue ? quilt_queue_bytes(a.q_block) : 0);
  const unsigned g = (unsigned)((a.q_bands + 7) / 8) * 8u * (unsigned)a.q_subsets;
  quilt_kernel(a.tm != nullptr, a.q_queue, a.q_block)<<<g, a.q_block, lds, s>>>(a);
  // the error stays set for callers that check it after the frame's launches
  return hipPeekAtLastError();
}

void launch_interleave(const InterleaveArgs& a, hipStream_t s) {
  const uint32_t per_row = nblk(a.Wp, 256 * 4);
  const uint32_t nb = per_row * (uint32_t)a.Hp;
  const int64_t plane = 4ll * a.Wv * a.Hv;
  if (plane < (1 << 24) && plane * a.V < (1ll << 32)) {
    if (a.mode == 0) k_interleave_small<1><<<nb, 256, 0, s>>>(a, per_row, nb);
    else k_interleave_small<8><<<nb, 256, 0, s>>>(a, per_row, nb);
  } else {
    k_interleave<<<nb, 256, 0, s>>>(a, per_row, nb);
  }
}

void launch_angular_filter(const AngularArgs& a, hipStream_t s) {
  dim3 g(nblk(((int64_t)a.W * a.H + 3) / 4, 256), (unsigned)a.V);
  k_angular_filter<<<g, 256, 0, s>>>(a);
}

}  // namespace lfdpr
