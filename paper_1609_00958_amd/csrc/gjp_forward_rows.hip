// gjp_forward_rows.hip -- forward of the generalized Joseph projector for
// column geometries (every view's dv parallel to axis 2, no ray driven by axis
// 2), straight from the caller's volume: no padded copies.
//
// All rays v of a detector column u share the driving axis m and the in-plane
// line p_a(i) = s_a + (i - s_m) g_a, so on plane i they interpolate between the
// same two voxel rows; their axis-2 coordinates are A + v B. A wavefront takes
// 64 RPL rays of one column. Per plane it reads the piece of the two rows that
// its rays span with coalesced 16-byte loads (lane = four voxels), combines them
// with the plane's in-plane weights and leaves the combined row in LDS; each lane
// then interpolates its rays from one LDS read of two neighbours each. The
// bilinear weights of Eqs. 10-12 are applied row first, as two factors.
//
// Why: reading the four neighbours of every ray from memory instead takes an
// irregular 16-byte load per sample (two per three samples where three rays of a
// lane share them), which the address unit serves at four lanes per clock, and
// two padded copies of the volume per call. Coalesced rows cost 32 bytes per
// voxel row pair and 64 RPL rays. What bounds the kernel: the vector ALUs and the
// vector memory path together. At 512^3, 720 views of 768^2 a sample takes 12.4
// instructions, seven of its own (three of half rate) and the rest its share of the
// plane's; at two cycles each they fill 55% of the ALUs' time, at the rates measured
// for them one by one 75-90%. The data unit is busy 98% of the time (a quarter of
// it waiting for L1: the rows come from L2, since the wavefronts of neighbouring
// columns drift apart), the address unit 87%, LDS 62%. BF16, with half the bytes: 62,
// 98, 83 and 59%, and 56 instead of 60.5 ms.
// Measured steps, 256^3 / 360 views of 384^2: 4- and 8-byte loads 4.2 ms (the
// return path gives 30 bytes per clock whatever their width below 16), 16-byte
// loads 3.7 ms, the next planes' loads issued before the current ones are
// sampled and all LDS reads of a plane before its sums 3.3 ms.
// Copies' kernel -> this one, uniform random volumes: 256^3 as above 5.7 -> 3.4 ms,
// 512^3 / 720 views of 768^2 76.8 -> 60.7 ms (its three-rays-per-lane tiles; 95 ms
// with one), 1024^3 BF16 / 120 views of 1536^2 115 -> 93 ms, 64^3 / 64 views 29 -> 22
// us. A phantom that is half zeros takes 54 ms at 512^3 (likely the power limit).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gjp_internal.h"

namespace gjp {

struct bf16_t {
  uint16_t bits;
};
struct f16_t {
  uint16_t bits;
};

namespace {

constexpr int kSub = kRowPlanes;
constexpr int kRow = kRowEntries;  // a combined row in LDS: voxels, and zeros beside the grid
// How a window's voxels are read: a piece of 256, four voxels per lane; the same
// and one more voxel per lane (384 rays at magnification 1.5 span up to 290); two
// such pieces.
enum Window { ONE_PIECE, AND_TAIL, TWO_PIECES };
// Planes that a wavefront loads together, while it combines and samples as many
// earlier ones: two where the registers of four wavefronts per SIMD allow it (six
// rays per lane spill with two: 3.55 instead of 3.38 ms at 256^3, 360 views).
constexpr int planes_together(int window, int rpl) {
  return window == ONE_PIECE && rpl < 6 ? 2 : 1;
}
static_assert(kRowStep % (2 * planes_together(ONE_PIECE, 2)) == 0 && kRowStep % 2 == 0,
              "row_planes covers the planes that the loop takes");
constexpr uint32_t kNoLower = 0x80000000u, kNoUpper = 1u;  // offsets are even and below 2^31

// Four neighbouring elements of a row; 16-bit rows start on 4 bytes.
typedef uint32_t u2v __attribute__((ext_vector_type(2)));
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef _Float16 h4v __attribute__((ext_vector_type(4)));
template <typename T>
struct Four {
  typename std::conditional<sizeof(T) == 4, u4v, u2v>::type v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff) {
    if constexpr (sizeof(T) == 4)
      v = __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, soff, 0));
    else
      v = __builtin_bit_cast(u2v, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0));
  }
  __device__ __forceinline__ f4v get() const {
    if constexpr (sizeof(T) == 4) {
      return __builtin_bit_cast(f4v, v);
    } else if constexpr (std::is_same<T, bf16_t>::value) {
      return f4v{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                 __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
    } else {
      const h4v h = __builtin_bit_cast(h4v, v);
      return f4v{(float)h.x, (float)h.y, (float)h.z, (float)h.w};
    }
  }
};

// One element.
template <typename T>
struct One {
  uint32_t v;
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t rs, uint32_t voff, uint32_t soff) {
    if constexpr (sizeof(T) == 4)
      v = __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0);
    else
      v = __builtin_amdgcn_raw_buffer_load_b16(rs, voff, soff, 0);
  }
  __device__ __forceinline__ float get() const {
    if constexpr (sizeof(T) == 4)
      return __uint_as_float(v);
    else if constexpr (std::is_same<T, bf16_t>::value)
      return __uint_as_float(v << 16);
    else
      return (float)__builtin_bit_cast(_Float16, (uint16_t)v);
  }
};

__device__ __forceinline__ int wave_min(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
  return v;
}

__device__ __forceinline__ int floor_int(float p) {
  int i;
  asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(i) : "v"(p));
  return i;
}

// Weight of the upper neighbour at fraction d.
template <int WF>
__device__ __forceinline__ float upper(float d) {
  if constexpr (WF == W_SPLINE)
    return d * d * __builtin_fmaf(-2.0f, d, 3.0f);
  else
    return d;
}

typedef float f4l __attribute__((ext_vector_type(4), may_alias));

// The value, computed anew where it is used (keeps the compiler from carrying
// one address per plane and ray).
__device__ __forceinline__ uint32_t here_u(uint32_t x) {
  x = (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
  asm("" : "+s"(x));
  return x;
}

struct RowsShared {
  float row[2 * kRow];  // combined rows of a group of planes
  float2 w[64];         // in-plane weights of 64 planes
};
typedef __attribute__((address_space(3))) float lds_float;

// The volume from `base` on, `size` bytes; with size 0 every load returns zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer(const char* base, uint32_t size) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), (short)0, (int)size, 0x00020000);
}

// Planes j .. j + np - 1 of the wavefront's block (off: byte offset of a plane's
// lower row, one plane per lane, with kNoLower and kNoUpper where that row is
// absent and reads as zero; Sa: bytes to the row above it). The window's voxels
// zd .. zd + need - 1 go to entries pad, pad + 1, ... of the LDS rows, whose other
// entries are not touched. Rays lie p = fi gb + cb voxels above voxel zd (p >= -pad;
// kept small on the grid, for the precision of its fraction), fi counted from
// plane j.
template <typename T, int WF, int RPL, int WIN>
__device__ __forceinline__ void project_planes(const char* vol, uint32_t size, int zd, int need,
                                               int pad, int n2, uint32_t Sa, int off, int j, int np,
                                               RowsShared& sh, int lane, const float* gb,
                                               const float* cb, float* acc) {
  constexpr int G = planes_together(WIN, RPL), NP = WIN == TWO_PIECES ? 2 : 1;
  // byte offsets of the lane's voxels; off the window: beyond the buffer, reads zero
  uint32_t vo[NP], vt = 0;
#pragma unroll
  for (int c = 0; c < NP; ++c) {
    const int k = 256 * c + 4 * lane;
    vo[c] = k < need ? (uint32_t)(zd + k) * (uint32_t)sizeof(T) : 0x80000000u;
  }
  if (WIN == AND_TAIL) {
    vt = 256 + lane < need ? (uint32_t)(zd + 256 + lane) * (uint32_t)sizeof(T) : 0x80000000u;
  }
  struct Rows {
    Four<T> lo[G][NP], up[G][NP];
    One<T> tail_lo[G], tail_up[G];
  };
  const auto load = [&](Rows& x, int j) {
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane(off, j + k);
      const __amdgpu_buffer_rsrc_t lower = buffer(vol, o & kNoLower ? 0u : size);
      const __amdgpu_buffer_rsrc_t above = buffer(vol, o & kNoUpper ? 0u : size);
      const uint32_t so = o & ~(kNoLower | kNoUpper);
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        x.lo[k][c].load(lower, vo[c], so);
        x.up[k][c].load(above, vo[c], so + Sa);
      }
      if (WIN == AND_TAIL) {
        x.tail_lo[k].load(lower, vt, so);
        x.tail_up[k].load(above, vt, so + Sa);
      }
    }
  };
  float* const row = sh.row + pad;
  const auto sample = [&](const Rows& x, int j, float fi) {
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const float2 w = sh.w[j + k];
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        const f4v lo = x.lo[k][c].get(), up = x.up[k][c].get();
        f4l e = {__builtin_fmaf(w.y, up.x, w.x * lo.x), __builtin_fmaf(w.y, up.y, w.x * lo.y),
                 __builtin_fmaf(w.y, up.z, w.x * lo.z), __builtin_fmaf(w.y, up.w, w.x * lo.w)};
        if (n2 & 3) {  // the last four of a row may reach past its end
          const int z = zd + 256 * c + 4 * lane;
          e.y = z + 1 < n2 ? e.y : 0.0f;
          e.z = z + 2 < n2 ? e.z : 0.0f;
          e.w = z + 3 < n2 ? e.w : 0.0f;
        }
        if (256 * c + 4 * lane < need)
          *reinterpret_cast<f4l*>(row + k * kRow + 256 * c + 4 * lane) = e;
      }
      if (WIN == AND_TAIL && 256 + lane < need)
        row[k * kRow + 256 + lane] = __builtin_fmaf(w.y, x.tail_up[k].get(), w.x * x.tail_lo[k].get());
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < G; ++k) {
      const uint32_t at = here_u((uint32_t)(uintptr_t)(lds_float*)(row + k * kRow));
      float w[RPL], e0[RPL], e1[RPL];
#pragma unroll
      for (int r = 0; r < RPL; ++r) {
        const float p = __builtin_fmaf(fi + (float)k, gb[r], cb[r]);
        const lds_float* e = (const lds_float*)(uintptr_t)(at + 4u * (uint32_t)floor_int(p));
        e0[r] = e[0];
        e1[r] = e[1];
        w[r] = upper<WF>(__builtin_amdgcn_fractf(p));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int r = 0; r < RPL; ++r)
        acc[r] = __builtin_fmaf(w[r], e1[r], __builtin_fmaf(1.0f - w[r], e0[r], acc[r]));
    }
    __builtin_amdgcn_wave_barrier();
  };
  // (no branch around a load: its waits would then cover every load)
  Rows x, y;
  load(x, j);
  float fi = 0.0f;
  for (; np > 2 * G; np -= 2 * G) {
    load(y, j + G);
    __builtin_amdgcn_sched_barrier(0);
    sample(x, j, fi);
    load(x, j + 2 * G);
    __builtin_amdgcn_sched_barrier(0);
    sample(y, j + G, fi + (float)G);
    j += 2 * G;
    fi += (float)(2 * G);
  }
  load(y, j + G);
  __builtin_amdgcn_sched_barrier(0);
  sample(x, j, fi);
  sample(y, j + G, fi + (float)G);
}

// Rays v0 .. v0 + 64 RPL - 1 of column u of a view.
template <typename T, int WF, int RPL>
__device__ __forceinline__ void project_column(const FwdArgs& a, const void* volume, int view, int u, int v0,
                                               RowsShared& sh) {
  const int lane = threadIdx.x & 63;
  const double* v = a.views + 12 * (size_t)view;
  const bool cone = a.G.beam == BEAM_CONE;
  // the column's line (ray_line's arithmetic; dv_0 = dv_1 = 0)
  const double du = (double)u;
  const double d0 = v[3] + du * v[6], d1 = v[4] + du * v[7], d2 = v[5] + du * v[8];
  const double s0 = cone ? v[0] : d0, s1 = cone ? v[1] : d1;
  const double r0 = cone ? d0 - v[0] : v[0], r1 = cone ? d1 - v[1] : v[1];
  const bool m1 = fabs(r1) > fabs(r0);
  const double sm = m1 ? s1 : s0, sa = m1 ? s0 : s1, rm = m1 ? r1 : r0, ra = m1 ? r0 : r1;
  const int nm = m1 ? a.G.n[1] : a.G.n[0], na = m1 ? a.G.n[0] : a.G.n[1], n2 = a.G.n[2];
  const int last = min(a.n_v - v0, 64 * RPL) - 1;  // last ray of the wavefront
  float acc[RPL];
#pragma unroll
  for (int r = 0; r < RPL; ++r) acc[r] = 0.0f;
  const double irm = 1.0 / rm, ga = ra / rm;
  // axis-2 coordinate of ray v0 + k on plane i: (A + k B) + (i - sm) (C + k D)
  const double A = (cone ? v[2] : d2 + (double)v0 * v[11]);
  const double B = cone ? 0.0 : v[11];
  const double C = (cone ? d2 + (double)v0 * v[11] - v[2] : v[2]) * irm;
  const double D = cone ? v[11] * irm : 0.0;
  if (rm != 0.0) {
    // planes where the line is inside the padded grid (a little more; planes
    // outside weigh zero)
    double lo = 0.0, hi = (double)nm;
    if (ga != 0.0) {
      const double e0 = sm + (-1.0 - sa) / ga, e1 = sm + ((double)na - sa) / ga;
      lo = fmax(lo, fmin(e0, e1) - 0.5);
      hi = fmin(hi, fmax(e0, e1) + 1.5);
    } else if (!(sa > -1.0 && sa < (double)na)) {
      hi = lo;
    }
    const int i_lo = __builtin_amdgcn_readfirstlane((int)fmin(lo, (double)nm));
    const int i_hi = __builtin_amdgcn_readfirstlane((int)fmax(hi, 0.0));
    const uint64_t Sm = (uint64_t)(m1 ? 1 : a.G.n[1]) * (uint64_t)n2 * sizeof(T);
    const uint64_t Sa = (uint64_t)(m1 ? a.G.n[1] : 1) * (uint64_t)n2 * sizeof(T);
    const uint64_t total = (uint64_t)a.G.n[0] * a.G.n[1] * n2 * sizeof(T);
    for (int base = i_lo; base < i_hi; base += 64) {
      // lane l: plane base + l
      const int plane = base + lane;
      const double pa = sa + (-sm + (double)plane) * ga;
      const double fl = floor(pa);
      bool ok = plane < i_hi && pa > -1.0 && pa < (double)na;
      if (a.G.clip) {
        const double dx = (m1 ? pa : (double)plane) - a.G.cyl[0];
        const double dy = (m1 ? (double)plane : pa) - a.G.cyl[1];
        ok = ok && dx * dx + dy * dy < a.G.cyl_r2;
      }
      const int row = (int)fl;  // -1 .. na - 1
      const float wu = upper<WF>((float)(pa - fl)), wl = 1.0f - wu;
      sh.w[lane] = ok ? make_float2(wl, wu) : make_float2(0.0f, 0.0f);
      const int rmin = __builtin_amdgcn_readfirstlane(wave_min(ok ? row : 0x7fffffff));
      if (rmin == 0x7fffffff) continue;  // no plane of the block has samples
      const uint32_t at = (uint32_t)((uint64_t)lane * Sm + (uint64_t)(row - rmin) * Sa);
      const int off = (int)(!ok ? kNoLower | kNoUpper
                                : at | (row < 0 ? kNoLower : 0u) | (row + 1 < na ? 0u : kNoUpper));
      // the block's first byte (before the volume, and not read, where row -1 is
      // a lower one) and the bytes that its offsets reach
      const int64_t org = (int64_t)base * (int64_t)Sm + (int64_t)rmin * (int64_t)Sa;
      const char* vol = static_cast<const char*>(volume) + org;
      const uint32_t size = (uint32_t)min((int64_t)total - org, (int64_t)0x7fffffff);
      const int cnt = min(64, i_hi - base);
      for (int j = 0; j < cnt; j += kSub) {
        // window of voxels that the rays span on the planes that the loop takes (up to
        // three past the last one's, whose rows read as zeros)
        const double t0 = (double)(base + j) - sm;
        RowWindow win;
        if (!row_window(A, B, C, D, t0, row_planes(min(kSub, cnt - j)), last, n2, win)) continue;
        const int zd = __builtin_amdgcn_readfirstlane(win.zd);
        const int need = __builtin_amdgcn_readfirstlane(win.need);
        const int pad = __builtin_amdgcn_readfirstlane(win.pad);
        if (win.border) {  // beside the grid: zeros
#pragma unroll
          for (int k = 0; k < 2 * kRow / 256; ++k)
            reinterpret_cast<f4l*>(sh.row)[64 * k + lane] = f4l{0.0f, 0.0f, 0.0f, 0.0f};
        }
        // (not kept from the window on: one scalar register too many, and FP16 with two
        // rays per lane passed 96 vector registers, four instead of five wavefronts)
        const int np = min(kSub, (int)here_u((uint32_t)cnt) - j);
        float gb[RPL], cb[RPL];
#pragma unroll
        for (int r = 0; r < RPL; ++r) {
          const double k = (double)min(64 * r + lane, last);
          const double g = C + k * D;
          gb[r] = (float)g;
          cb[r] = (float)(A + k * B + t0 * g - (double)zd);
        }
        if (need <= 256)
          project_planes<T, WF, RPL, ONE_PIECE>(vol, size, zd, need, pad, n2, (uint32_t)Sa,
                                                 off, j, np, sh, lane, gb, cb, acc);
        else if (need <= 320)
          project_planes<T, WF, RPL, AND_TAIL>(vol, size, zd, need, pad, n2, (uint32_t)Sa,
                                                 off, j, np, sh, lane, gb, cb, acc);
        else
          project_planes<T, WF, RPL, TWO_PIECES>(vol, size, zd, need, pad, n2, (uint32_t)Sa,
                                                 off, j, np, sh, lane, gb, cb, acc);
      }
    }
  }
  const double wa = ga * (m1 ? a.G.vs[0] : a.G.vs[1]), wm = m1 ? a.G.vs[1] : a.G.vs[0];
  float* out = a.sino + ((size_t)view * a.n_u + u) * a.n_v + v0;
#pragma unroll
  for (int r = 0; r < RPL; ++r) {
    const int k = 64 * r + lane;
    const double g = (C + (double)k * D) * a.G.vs[2];
    if (k <= last)
      out[k] = rm != 0.0 ? acc[r] * __builtin_sqrtf((float)(wa * wa + wm * wm + g * g)) : 0.0f;
  }
}

// Tile `tile` of a view: four columns, 64 RPL rays.
template <typename T, int WF, int RPL>
__device__ __forceinline__ void project_tile(const FwdArgs& a, const void* volume, int view,
                                             int tile, RowsShared* sh) {
  const int tv = tile / a.tiles_u, tu = tile - tv * a.tiles_u;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int u = tu * 4 + wave;
  if (u < a.n_u) project_column<T, WF, RPL>(a, volume, view, u, tv * 64 * RPL, sh[wave]);
}

// Launch order: as fwd_kernel's (groups of view_group views; per group, tiles of
// four columns column group by column group along one band of rays, each tile
// for the group's views in turn), XCDs walking contiguous ranges.
template <typename T, int WF, int RPL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void fwd_rows_kernel(
    const FwdArgs a) {
  __shared__ __align__(16) RowsShared sh[4];
  const uint32_t nb = gridDim.x;
  const uint32_t b = (blockIdx.x % 8) * (nb / 8) + min(blockIdx.x % 8, nb % 8) + blockIdx.x / 8;
  const uint32_t K = (uint32_t)a.view_group, tpv = (uint32_t)a.tiles_per_view;
  const uint32_t grp = b / (K * tpv);
  const uint32_t r = b - grp * K * tpv;
  const uint32_t v0 = grp * K;
  const uint32_t kg = min(K, (uint32_t)a.n_views - v0);  // views in this group
  const uint32_t t = r / kg;
  project_tile<T, WF, RPL>(a, a.vol, (int)(v0 + (r - t * kg)), (int)t, sh);
}

// Persistent batched forward of the row-forward instances of one storage type
// and weight, whatever their rays per lane: queues, items and exit as in
// batched_loop (gjp_kernels.hip).
template <typename T, int WF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void batched_rows_kernel(
    const BatchInst* __restrict__ insts, const uint2* __restrict__ items,
    const int* __restrict__ qoff, int* __restrict__ counters) {
  __shared__ __align__(16) RowsShared sh[4];
  __shared__ int s_item;
  const int home = (int)(blockIdx.x % kBatchQueues);
  for (int d = 0; d < kBatchQueues; ++d) {
    const int q = (home + d) % kBatchQueues;
    const int begin = qoff[q], n = qoff[q + 1] - begin;
    for (;;) {
      if (threadIdx.x == 0) s_item = atomicAdd(&counters[q], 1);
      __syncthreads();
      const int item = __builtin_amdgcn_readfirstlane(s_item);
      __syncthreads();
      if (item >= n) break;
      const uint2 it = items[begin + item];
      const BatchInst& I = insts[__builtin_amdgcn_readfirstlane((int)(it.x & 0xfffu))];
      const int view = __builtin_amdgcn_readfirstlane((int)(it.x >> 12));
      const int tile = __builtin_amdgcn_readfirstlane((int)it.y);
      switch (I.a.rows) {
        case 2: project_tile<T, WF, 2>(I.a, I.src, view, tile, sh); break;
        case 3: project_tile<T, WF, 3>(I.a, I.src, view, tile, sh); break;
        case 4: project_tile<T, WF, 4>(I.a, I.src, view, tile, sh); break;
        default: project_tile<T, WF, 6>(I.a, I.src, view, tile, sh); break;
      }
    }
  }
}

template <typename T, int WF>
void launch_rows_t(const FwdArgs& a, unsigned grid, hipStream_t s) {
  switch (a.rows) {
    case 2: fwd_rows_kernel<T, WF, 2><<<grid, 256, 0, s>>>(a); break;
    case 3: fwd_rows_kernel<T, WF, 3><<<grid, 256, 0, s>>>(a); break;
    case 4: fwd_rows_kernel<T, WF, 4><<<grid, 256, 0, s>>>(a); break;
    default: fwd_rows_kernel<T, WF, 6><<<grid, 256, 0, s>>>(a); break;
  }
}
template <typename T>
void launch_rows_w(const FwdArgs& a, int weight, unsigned grid, hipStream_t s) {
  if (weight == W_SPLINE)
    launch_rows_t<T, W_SPLINE>(a, grid, s);
  else
    launch_rows_t<T, W_LINEAR>(a, grid, s);
}

using BatchedRows = void (*)(const BatchInst*, const uint2*, const int*, int*);
BatchedRows batched_rows_kernel_of(int dtype, int weight) {
  const bool spline = weight == W_SPLINE;
  if (dtype == 0)
    return spline ? batched_rows_kernel<float, W_SPLINE> : batched_rows_kernel<float, W_LINEAR>;
  if (dtype == 1)
    return spline ? batched_rows_kernel<bf16_t, W_SPLINE> : batched_rows_kernel<bf16_t, W_LINEAR>;
  return spline ? batched_rows_kernel<f16_t, W_SPLINE> : batched_rows_kernel<f16_t, W_LINEAR>;
}

}  // namespace

void launch_forward_rows(const FwdArgs& a, int dtype, int weight, unsigned grid, hipStream_t s) {
  if (dtype == 0)
    launch_rows_w<float>(a, weight, grid, s);
  else if (dtype == 1)
    launch_rows_w<bf16_t>(a, weight, grid, s);
  else
    launch_rows_w<f16_t>(a, weight, grid, s);
}

const void* batched_rows_function(int dtype, int weight) {
  return reinterpret_cast<const void*>(batched_rows_kernel_of(dtype, weight));
}

void launch_batched_rows(const BatchInst* d_insts, const uint2* d_items, const int* d_qoff,
                         int* d_counters, int grid, int dtype, int weight, hipStream_t s) {
  batched_rows_kernel_of(dtype, weight)<<<grid, 256, 0, s>>>(d_insts, d_items, d_qoff, d_counters);
}

}  // namespace gjp
