// gjp_adjoint_free.hip -- adjoint of the generalized Joseph projector for
// general geometries (detectors in any position, every driving axis): voxels
// gather the samples that touch them.
//
// A workgroup owns a tile of 16 x 16 x 8 voxels, a lane a cube of 2 x 2 x 2 of
// them, whose sums stay in registers over all views. Per view and driving axis m
// the rays that can touch the tile form a rectangle of the detector (the
// perspective image of the tile grown by one voxel in the two other directions);
// the workgroup stages them in LDS as lines p(i) = p_0 + i g relative to the tile,
// and every lane walks the few of them whose detector position is near its cube's:
// the image of the cube grown by one voxel lies within half extents (hu, hv) of
// the image of its centre, which are bounded once per tile, so all lanes walk the
// same number of rays, nu x nv. Each ray is read from LDS once for the cube's two
// planes and, per plane, its four voxels.
//
// Why: spreading each sample to its four voxels with LDS additions instead costs
// four read-modify-writes per sample, for rays that mostly miss the tile's planes,
// and stages every ray for the whole tile. What bounds the gather: the vector ALUs
// (200 M wavefront instructions, 56% of the time at two cycles each and about 85% at
// the rates measured for them, for 120 x 136 x 112 voxels and 48 views of 180 x 200; a
// ray takes 30 per cube, and five in six of the rays walked have no weight in a given
// voxel); LDS is 34% busy. Spread -> gather, with the ray table: that case 2.3 -> 0.36
// ms; 40^3, 16 views of 44^2 378 -> 71 us; 64^3, 32 views of 200^2 4.98 -> 0.18 ms;
// 160^3, 60 views of 250^2 3.10 -> 0.89 ms.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "gjp_internal.h"

namespace gjp {
namespace {

constexpr int TX = 16, TY = 16, TZ = 8;  // voxels of a tile: four wavefronts of 8 x 8 x 8
constexpr int kRays = 2000;              // staged rays (40 kB: four workgroups per CU)

struct FreeArgs {
  int n[3], n_u, n_v;
  const float* proj;    // 12 floats per view (launch_adjoint_gather)
  const float4* table;  // adj_table_kernel's, 32 bytes per ray
  const int* mask;      // driving axes per view
  int n_views, accumulate;
  float* out;    // volume, or one partial volume per split
  size_t slice;  // floats between partial volumes
};

struct Staged {
  float4 line[kRays];  // p_a and g_a, p_b and g_b on the tile's first plane
  float val[kRays];    // 0: not a ray of this axis
  int bad;             // a value is not finite
};

// 1 - |x|, or 0 beyond.
template <int WF>
__device__ __forceinline__ float tent(float x) {
  float r;
  asm("v_sub_f32_e64 %0, 1.0, |%1| clamp" : "=v"(r) : "v"(x));
  if constexpr (WF == W_SPLINE) r = r * r * __builtin_fmaf(-2.0f, r, 3.0f);
  return r;
}

// One ray's samples on two planes for a cube: acc[4 x + 2 y + z]. CHECK: values
// that are not finite reach only the voxels that they have weight in.
template <int WF, int M, bool CHECK>
__device__ __forceinline__ void add_ray(const float4 e, float y, float fm, float fa, float fb,
                                        float* acc) {
  constexpr int sm = M == 0 ? 4 : M == 1 ? 2 : 1, sa = M == 0 ? 2 : 4, sb = M == 2 ? 2 : 1;
  float a = __builtin_fmaf(fm, e.y, e.x) - fa, b = __builtin_fmaf(fm, e.w, e.z) - fb;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float wa[2] = {tent<WF>(a), tent<WF>(a - 1.0f)};
    const float wb[2] = {tent<WF>(b), tent<WF>(b - 1.0f)};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const float p = !CHECK || wb[k] > 0.0f ? y * wb[k] : 0.0f;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        float& s = acc[i * sm + j * sa + k * sb];
        if (!CHECK || wa[j] > 0.0f) s = __builtin_fmaf(wa[j], p, s);
      }
    }
    a += e.y;
    b += e.w;
  }
}

// Largest |d num / w| for moves of at most (dx, dy, dz) from points whose
// coordinate num / w lies in [lo, hi], w >= wmin at the end.
__device__ __forceinline__ float half_extent(const float* num, const float* den, float lo, float hi,
                                             float dx, float dy, float dz, float inv_wmin) {
  const auto m = [&](int k) {
    return fmaxf(__builtin_fabsf(num[k] - lo * den[k]), __builtin_fabsf(num[k] - hi * den[k]));
  };
  return (dx * m(0) + dy * m(1) + dz * m(2)) * inv_wmin + 0.02f;
}

__device__ __forceinline__ float uniform(float x) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x)));
}

template <int WF, int M>
__device__ __forceinline__ void gather_axis(const FreeArgs& a, const float4* T, const int* o,
                                            int wu0, int wv0, int nwu, int nwv, int nu, int nv,
                                            int u0, int v0, int cm, int ca, int cb, Staged& sh,
                                            float* acc) {
  const float om = (float)o[M], oa = (float)o[M == 0 ? 1 : 0], ob = (float)o[M == 2 ? 1 : 2];
  const float fm = (float)cm, fa = (float)ca, fb = (float)cb;
  // parts of the rectangle that fit (mostly the whole): columns, rays of a column
  const int pv = min(nwv, kRays), pu = min(nwu, kRays / pv);
  for (int q = 0; q < nwu; q += pu)
    for (int r = 0; r < nwv; r += pv) {
      const int cu = min(pu, nwu - q), cv = min(pv, nwv - r), n = cu * cv;
      const float inv = 1.0f / (float)cv;
      bool bad = false;
      for (int k = threadIdx.x; k < n; k += 256) {
        int ku = (int)((float)k * inv);  // k / cv (k < 2000: off by at most one)
        int kv = k - ku * cv;
        if (kv < 0) { --ku; kv += cv; }
        if (kv >= cv) { ++ku; kv -= cv; }
        const int iu = wu0 + q + ku, iv = wv0 + r + kv;
        float4 line = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        float val = 0.0f;
        // (always; without the test 22.6 instead of 21.6 ms for 60^3, 8 views of 1500^2)
        if (iu < a.n_u && iv < a.n_v) {
          const float4* e = T + 2 * ((size_t)iu * a.n_v + iv);
          const float4 e0 = e[0];
          const float2 e1 = *reinterpret_cast<const float2*>(e + 1);
          const uint32_t mr = __float_as_uint(e0.x);
          if ((int)(mr & 3u) == M && (mr >> 17) > ((mr >> 2) & 0x7fffu)) {
            line = make_float4(__builtin_fmaf(om, e0.z, e0.y) - oa, e0.z,
                               __builtin_fmaf(om, e1.x, e0.w) - ob, e1.x);
            val = e1.y;
          }
        }
        sh.line[k] = line;
        sh.val[k] = val;
        bad = bad || !(__builtin_fabsf(val) < 3.0e38f);
      }
      if (bad) sh.bad = 1;
      __syncthreads();
      const bool check = __builtin_amdgcn_readfirstlane(sh.bad) != 0;
      if (!check && cu == nwu && cv == nwv) {
        int at = (u0 - wu0) * cv + (v0 - wv0);
        for (int ku = 0; ku < nu; ++ku, at += cv)
          for (int kv = 0; kv < nv; ++kv)
            add_ray<WF, M, false>(sh.line[at + kv], sh.val[at + kv], fm, fa, fb, acc);
      } else {
        const int bu = u0 - wu0 - q, bv = v0 - wv0 - r;
        for (int ku = max(bu, 0); ku < min(bu + nu, cu); ++ku)
          for (int kv = max(bv, 0); kv < min(bv + nv, cv); ++kv)
            add_ray<WF, M, true>(sh.line[ku * cv + kv], sh.val[ku * cv + kv], fm, fa, fb, acc);
      }
      __syncthreads();
      if (check) {
        sh.bad = 0;
        __syncthreads();
      }
    }
}

template <int WF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void adj_free_kernel(
    const FreeArgs a) {
  __shared__ Staged sh;
  const int nty = (a.n[1] + TY - 1) / TY, ntz = (a.n[2] + TZ - 1) / TZ;
  // tiles along axis 2 first, XCDs walking contiguous ranges
  const uint32_t nb = gridDim.x;
  const uint32_t b = (blockIdx.x % 8) * (nb / 8) + min(blockIdx.x % 8, nb % 8) + blockIdx.x / 8;
  const int tz = (int)(b % (uint32_t)ntz), ty = (int)(b / (uint32_t)ntz % (uint32_t)nty),
            tx = (int)(b / (uint32_t)ntz / (uint32_t)nty);
  const int o[3] = {tx * TX, ty * TY, tz * TZ};
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the lane's cube, relative to the tile
  const int cx = 8 * (wave & 1) + 2 * (lane >> 4), cy = 8 * (wave >> 1) + 2 * ((lane >> 2) & 3),
            cz = 2 * (lane & 3);
  // range of the cubes' centres (cubes outside the grid: moved into it, not written)
  float lo[3], hi[3], c[3];
  const int T[3] = {TX, TY, TZ}, cc[3] = {cx, cy, cz};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lo[k] = (float)o[k] + 0.5f;
    hi[k] = (float)min(o[k] + T[k] - 2, a.n[k] - 1) + 0.5f;
    c[k] = fminf(lo[k] + (float)cc[k], hi[k]);
  }
  float acc[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
  if (threadIdx.x == 0) sh.bad = 0;
  __syncthreads();
  const int view0 = (int)((long long)a.n_views * blockIdx.y / gridDim.y);
  const int view1 = (int)((long long)a.n_views * (blockIdx.y + 1) / gridDim.y);
  for (int view = view0; view < view1; ++view) {
    const int mk = a.mask[view];
    if (!mk) continue;
    const float* P = a.proj + 12 * (size_t)view;
    const auto num = [&](int r, float x, float y, float z) {
      return __builtin_fmaf(P[4 * r], x, __builtin_fmaf(P[4 * r + 1], y,
                                                        __builtin_fmaf(P[4 * r + 2], z, P[4 * r + 3])));
    };
    // images of the corners of the centres' range, one per lane (mod 8)
    const float kx = lane & 1 ? hi[0] : lo[0], ky = lane & 2 ? hi[1] : lo[1],
                kz = lane & 4 ? hi[2] : lo[2];
    float w = num(2, kx, ky, kz);
    float ulo = num(0, kx, ky, kz) / w, vlo = num(1, kx, ky, kz) / w, uhi = ulo, vhi = vlo;
#pragma unroll
    for (int s = 1; s < 8; s *= 2) {
      w = fminf(w, __shfl_xor(w, s));
      ulo = fminf(ulo, __shfl_xor(ulo, s));
      uhi = fmaxf(uhi, __shfl_xor(uhi, s));
      vlo = fminf(vlo, __shfl_xor(vlo, s));
      vhi = fmaxf(vhi, __shfl_xor(vhi, s));
    }
    w = uniform(w) - 1.5f * (__builtin_fabsf(P[8]) + __builtin_fabsf(P[9]) + __builtin_fabsf(P[10]));
    ulo = uniform(ulo), uhi = uniform(uhi), vlo = uniform(vlo), vhi = uniform(vhi);
    const float inv_wmin = uniform(1.0f / w);
    const float inv = 1.0f / num(2, c[0], c[1], c[2]);
    const float uc = num(0, c[0], c[1], c[2]) * inv, vc = num(1, c[0], c[1], c[2]) * inv;
    const float4* rays = a.table + 2 * (size_t)view * a.n_u * a.n_v;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      if (!(mk >> m & 1)) continue;
      const float dx = m == 0 ? 0.5f : 1.5f, dy = m == 1 ? 0.5f : 1.5f, dz = m == 2 ? 0.5f : 1.5f;
      const float hu = uniform(half_extent(P, P + 8, ulo, uhi, dx, dy, dz, inv_wmin));
      const float hv = uniform(half_extent(P + 4, P + 8, vlo, vhi, dx, dy, dz, inv_wmin));
      const float fu = (float)a.n_u, fv = (float)a.n_v;
      // boxes that miss the detector altogether
      if (uhi + hu < -0.01f || vhi + hv < -0.01f || ulo - hu > fu - 0.99f || vlo - hv > fv - 0.99f)
        continue;
      // rays per lane: the integers of an interval of 2 h at most, and all of the
      // detector's where it is no longer than that
      const int nu = min(__builtin_amdgcn_readfirstlane((int)fminf(2.0f * hu, fu)) + 1, a.n_u);
      const int nv = min(__builtin_amdgcn_readfirstlane((int)fminf(2.0f * hv, fv)) + 1, a.n_v);
      // first rays of a lane and of all lanes. An interval that begins before the
      // detector, or has fewer than its count left on it, is moved onto it: what it
      // has there stays inside.
      const auto first = [](float x, int n, int count) {
        return min((int)fminf(fmaxf(ceilf(x), 0.0f), 1.0e9f), n - count);
      };
      const int wu0 = __builtin_amdgcn_readfirstlane(first(ulo - hu - 0.01f, a.n_u, nu));
      const int wv0 = __builtin_amdgcn_readfirstlane(first(vlo - hv - 0.01f, a.n_v, nv));
      const int wu1 = max(__builtin_amdgcn_readfirstlane(first(uhi - hu + 0.01f, a.n_u, nu)), wu0) + nu;
      const int wv1 = max(__builtin_amdgcn_readfirstlane(first(vhi - hv + 0.01f, a.n_v, nv)), wv0) + nv;
      const int u0 = min(max(first(uc - hu, a.n_u, nu), wu0), wu1 - nu);
      const int v0 = min(max(first(vc - hv, a.n_v, nv), wv0), wv1 - nv);
      if (m == 0)
        gather_axis<WF, 0>(a, rays, o, wu0, wv0, wu1 - wu0, wv1 - wv0, nu, nv, u0, v0, cx, cy, cz,
                           sh, acc);
      else if (m == 1)
        gather_axis<WF, 1>(a, rays, o, wu0, wv0, wu1 - wu0, wv1 - wv0, nu, nv, u0, v0, cy, cx, cz,
                           sh, acc);
      else
        gather_axis<WF, 2>(a, rays, o, wu0, wv0, wu1 - wu0, wv1 - wv0, nu, nv, u0, v0, cz, cx, cy,
                           sh, acc);
    }
  }
  float* out = a.out + (size_t)blockIdx.y * a.slice;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int x = o[0] + cx + (k >> 2), y = o[1] + cy + (k >> 1 & 1), z = o[2] + cz + (k & 1);
    if (x < a.n[0] && y < a.n[1] && z < a.n[2]) {
      const size_t i = ((size_t)x * a.n[1] + y) * a.n[2] + z;
      out[i] = a.accumulate ? out[i] + acc[k] : acc[k];
    }
  }
}

}  // namespace

int launch_adjoint_free(const gjp_geometry* g, const float* proj, const float4* table,
                        const int* mask, int n_views, bool accumulate, float* vol, float* part,
                        int splits, hipStream_t s) {
  FreeArgs a;
  for (int k = 0; k < 3; ++k) a.n[k] = g->n[k];
  a.n_u = g->n_u;
  a.n_v = g->n_v;
  a.proj = proj;
  a.table = table;
  a.mask = mask;
  a.n_views = n_views;
  a.accumulate = accumulate && splits <= 1 ? 1 : 0;
  a.out = splits > 1 ? part : vol;
  a.slice = (size_t)g->n[0] * g->n[1] * g->n[2];
  const unsigned long long tiles = (unsigned long long)((g->n[0] + TX - 1) / TX) *
                                   ((g->n[1] + TY - 1) / TY) * ((g->n[2] + TZ - 1) / TZ);
  if (tiles > 0x7fffffffull) return set_error(-4, "adjoint: volume too large for one launch");
  const dim3 grid((unsigned)tiles, (unsigned)(splits > 1 ? splits : 1));
  if (g->weight == W_SPLINE)
    adj_free_kernel<W_SPLINE><<<grid, 256, 0, s>>>(a);
  else
    adj_free_kernel<W_LINEAR><<<grid, 256, 0, s>>>(a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(-3, std::string("adjoint kernel: ") + hipGetErrorString(e));
  return splits > 1 ? launch_adjoint_sum(part, a.slice, splits, accumulate, vol, s) : 0;
}

}  // namespace gjp
