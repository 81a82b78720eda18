// gjp_adjoint_tiles.hip -- adjoint of the generalized Joseph projector for
// column geometries (every view's dv parallel to axis 2, no ray driven by axis
// 2).
//
// All rays v of detector column u share the driving axis m and the in-plane
// line p_a(i) = s_a + (i - s_m) g_a, and on plane i their axis-2 coordinates are
// A + v B. The adjoint of one plane therefore factors into a resampling of each
// column's rays along axis 2, s_u(z) = sum_v w(|A + v B - z|) y_uv, which does
// not depend on the in-plane row, and a spread over the two rows the column lies
// between on that plane, x(row, z) += w(|p_a(u) - row|) s_u(z). A wavefront owns
// one plane, R rows of it and 64 ZL voxels along axis 2 (lane = ZL neighbouring
// voxels): it resamples each column once, takes the columns cell by cell (the
// cell between two rows is known at compile time, so the rows stay in
// registers), and adds each to its two rows. A voxel-driven gather evaluates
// each column again for every block of rows it touches. (The spread as a
// 16 x 16 x 4 FP32 matrix product was slower: these instructions keep the vector
// unit of their SIMD idle for their 32 cycles, against 10 for the two rows.)
//
// A workgroup owns P planes; per view the detector window they need (columns u,
// rows v of the sinogram scaled by the rays' step lengths) is copied to LDS once
// and shared. The columns driven by axis 0 and by axis 1 are two launches, the
// second adding to the first's volume (one if the views have one of them only). For
// volumes whose tiles alone do not fill the device both axes and several splits of the
// views run as one launch into partial volumes, summed by a second kernel.
//
// What bounds it, at 512^3 / 720 views of 768^2: the vector ALUs (57% of the time at
// two cycles an instruction, about 75% at the rates measured for them) and LDS
// (80%, two fifths of it bank conflicts of the lanes' candidate reads).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gjp_internal.h"

namespace gjp {

namespace {

// Tile shape: 8 rows by 8 planes (wavefronts) keeps the accumulators within 64
// registers and four workgroups (eight wavefronts per SIMD) on a compute unit.
// 512^3 / 720 views / 768^2: 80 ms; 12 or 16 rows at six or four wavefronts per
// SIMD 91-99 ms, four voxels per lane 82 ms, staging double-buffered at four
// wavefronts per SIMD 87 ms.
constexpr int R = kTileEdge;
constexpr int P = kTileEdge;
constexpr int CH = 32;       // columns staged together at most
constexpr int kViews = 64;   // views whose windows are found together
constexpr int kRowPad = 12;  // entries after each staged column (candidate lists overrun its end)
constexpr int kFlip = 1 << 30;  // Window::kind: rows counted from the detector's other end
// Staged values (LDS words): what the other arrays leave of a quarter of 160 KB.
constexpr int CAP = (10240 - P * CH * 8 - 2 * (CH * 12 + 2) - kViews * 6 - 2 - 16) & ~3;
static_assert(CAP >= kTileMaxRows + kRowPad, "a window of kTileMaxRows rows fits");

struct TileArgs {
  GridGeom G;
  const double* views;
  const float* proj;
  const float* rays;  // y times step length, n_views x n_u x n_v
  float* vol;          // slice s of the launch: vol + s * slice
  size_t slice;
  int n_views, n_u, n_v;
  int m0;              // driving axis of slice 0; odd slices take the other one
  int both;            // 0: every slice takes m0
  int accumulate;      // add to vol (else overwrite it)
  int splits;          // slices 2 k and 2 k + 1 (both = 0: k): views k, k + splits, ...
  int nzb;             // tiles along axis 2
};

typedef __attribute__((address_space(3))) const float* lds_ptr;

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// The value, opaque to the compiler: what is computed from it stays where it is
// instead of being hoisted out of the view loop into registers.
__device__ __forceinline__ int here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
__device__ __forceinline__ int here_u(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

typedef uint32_t u4rsrc __attribute__((ext_vector_type(4)));

// LDS offset (bytes) of a shared-memory pointer; wave-uniform.
__device__ __forceinline__ uint32_t lds_offset(const float* p) {
  return (uint32_t)__builtin_amdgcn_readfirstlane(
      (int)(uintptr_t)(__attribute__((address_space(3))) const float*)p);
}

// One dword per active lane from byte offset off of a buffer (zero outside it)
// to LDS at dst + 4 lane, without a register. As assembly, because the compiler
// would otherwise make every later LDS read wait for it; the caller waits
// (vmcnt 0) before the barrier that publishes the data.
// Writes m0, which the compiler reserves and takes no clobber of: between save_m0 and
// restore_m0 only (around the loop and not in the block, which took 1% of the kernel).
__device__ __forceinline__ void load_to_lds(u4rsrc rs, uint32_t off, uint32_t dst) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 4\n\t"  // also covers scalar operands just written by vector instructions
      "buffer_load_dword %0, %1, 0 offen lds"
      :
      : "v"(off), "s"(rs), "s"(dst)
      : "memory");
}
__device__ __forceinline__ uint32_t save_m0() {
  uint32_t x;
  asm volatile("s_mov_b32 %0, m0" : "=s"(x));
  return x;
}
__device__ __forceinline__ void restore_m0(uint32_t x) { asm volatile("s_mov_b32 m0, %0" : : "s"(x)); }

__device__ __forceinline__ float clamp01(float x) { return __builtin_amdgcn_fmed3f(x, 0.0f, 1.0f); }

// min(max(a - b, 0), 1) in one full-rate instruction.
__device__ __forceinline__ float sub_clamp(float a, float b) {
  float r;
  asm("v_sub_f32_e64 %0, %1, %2 clamp" : "=v"(r) : "v"(a), "v"(b));
  return r;
}

// Weight of a sample at signed distance r (Eqs. 13, 14; zero from one voxel on).
template <int WF>
__device__ __forceinline__ float tent(float r) {
  if constexpr (WF == W_SPLINE) {
    const float t = fminf(__builtin_fabsf(r), 1.0f);
    return __builtin_fmaf(t * t, __builtin_fmaf(2.0f, t, -3.0f), 1.0f);
  } else {
    return clamp01(1.0f - __builtin_fabsf(r));
  }
}

// Columns of the staged chunk: the in-plane line p_a(i) = sa + (i - sm) ga of
// a column's rays and their axis-2 coordinates a0 + t a1 + v B (t = (i - sm)
// irm, v counted from the window's first row; irm = 0: not driven by the
// pass's axis).
struct Lines {
  double sm[CH], sa[CH], ga[CH], irm[CH], a0[CH], a1[CH];
  double dv;  // |dv| along axis 2
};

// A column on one wavefront's plane: ray k of the window lies at A + k (B + Bl)
// from the tile's first voxel along axis 2; w is the weight of the column's
// lower row and row the LDS address of its first staged value (less four times
// the rounding constant's bits).
struct Slot {
  float A, B, Bl, iB;
  float w;
  uint32_t row, pad[2];
};

// Detector window of a view on the tile: columns ulo .. uhi, nv rows from v0
// (rows may lie off the detector: they count as zeros), at most n candidate
// rays per voxel pair; kind: which fixed candidate list applies (0: none) (and
// kFlip).
struct Window {
  int ulo, uhi, v0, nv, n, kind;
};

// Candidate lists of N rays for the ZL voxels z .. z + ZL - 1 of a lane and ray
// spacings B in (lo, hi]: candidate i lies i B to (i + 1) B above z - 1, so that
// the list holds every ray within reach ((ZL + 1) / B <= N), and which weights
// can differ from zero, and on which side of their peak, is known per candidate.
template <int ZL, int N>
struct List {
  static constexpr double lo = (ZL + 1.0) / N + 0.0015;
  static constexpr double hi = N <= ZL + 1 ? 1.0e9 : (ZL + 1.0) / (N - 1.7);
};

// Calls f with each list length that has code of its own, shortest first.
template <int ZL, class F>
__device__ __forceinline__ void each_list(F f) {
  using std::integral_constant;
  f(integral_constant<int, ZL + 1>());
  f(integral_constant<int, ZL + 2>());
  f(integral_constant<int, ZL + 3>());
  f(integral_constant<int, ZL + 4>());
  if constexpr (ZL > 2) f(integral_constant<int, ZL + 5>());
  f(integral_constant<int, ZL == 1 ? 6 : (ZL == 2 ? 8 : 10)>());
}

template <int WF, int ZL>
__global__ __launch_bounds__(P * 64) __attribute__((amdgpu_waves_per_eu(8))) void adj_tile_kernel(const TileArgs a) {
  constexpr int ZT = 64 * ZL;  // voxels of a tile along axis 2
  __shared__ __align__(16) float s_buf[CAP];
  __shared__ __align__(16) Slot s_slot[P][CH];
  __shared__ Lines s_line[2];
  __shared__ Window s_win[kViews];
  __shared__ uint64_t s_mask;
  const int tid = threadIdx.x & 63;
  const int pl = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  Slot* slot = s_slot[pl];
  const int slice = blockIdx.y;
  const int m = a.m0 ^ (slice & a.both);

  // tile of this workgroup: XCDs walk contiguous ranges; within a block of
  // axis-2 tiles, strips of 8 tiles along the rows, so that the workgroups
  // resident on an XCD read the same few detector columns
  const uint32_t nb = gridDim.x;
  const uint32_t L = (blockIdx.x % 8) * (nb / 8) + min(blockIdx.x % 8, nb % 8) + blockIdx.x / 8;
  const int ntp = (a.G.n[m] + P - 1) / P, ntr = (a.G.n[1 - m] + R - 1) / R;
  const int per_z = ntp * ntr;
  const int zb = (int)(L / (uint32_t)per_z);
  if (zb >= a.nzb) return;  // the other axis's slices have more tiles
  const int q = (int)(L - (uint32_t)zb * per_z);
  const int strip = q / (8 * ntp);
  const int sw = min(8, ntr - 8 * strip);
  const int q2 = q - strip * 8 * ntp;
  const int tp = q2 / sw, tr = strip * 8 + (q2 - tp * sw);
  const int pm0 = tp * P, zt = zb * ZT;
  const int nm = a.G.n[m], na = a.G.n[1 - m], n2 = a.G.n[2];

  float acc[R][ZL];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int k = 0; k < ZL; ++k) acc[r][k] = 0.0f;

  const bool cone = a.G.beam == BEAM_CONE;
  // this slice's views: v0, v0 + splits, ...
  const int sv0 = slice >> a.both, ngv = (a.n_views - sv0 + a.splits - 1) / a.splits;
  bool store = a.accumulate == 0;

  for (int batch = 0; batch < ngv; batch += kViews) {
    __syncthreads();  // the previous batch's windows have been read, its sums stored
    if (pl == 0) {
      const int lane = here(tid), z0 = here_u(zt), ra0 = here_u(tr) * R;
      // windows of the slice's views batch .. batch + kViews - 1, one per lane
      const int gi = batch + lane;
      const int c = min(gi, ngv - 1) * a.splits + sv0;
      const double* v = a.views + 12 * (size_t)c;
      const TileWindow t = tile_window(v, a.proj + 12 * (size_t)c, cone, a.n_u, a.n_v, m, pm0, ra0,
                                       z0, ZT);
      const bool flip = v[11] < 0.0;  // rows counted from the other end
      const double bmin = t.bmin, bmax = t.bmax;
      Window w;
      w.ulo = t.ulo;
      w.uhi = t.uhi;
      // (the host has bounded the rows; the clamps only keep the window in LDS)
      w.v0 = (int)fmin(fmax(t.v0, -1.0e9), 1.0e9);
      w.nv = (int)fmin(fmax(t.v0 + t.rows - (double)w.v0, 1.0), (double)(CAP - kRowPad));
      w.n = (int)fmin(((double)ZL + 1.004) / bmin, 30000.0) + 1;
      w.kind = 0;
      auto offer = [&](auto n_) {
        constexpr int N = decltype(n_)::value;
        if (w.kind == 0 && bmin > List<ZL, N>::lo && bmax <= List<ZL, N>::hi) w.kind = N;
      };
      each_list<ZL>(offer);
      if (flip) w.kind |= kFlip;
      s_win[lane] = w;
      const uint64_t some =
          __ballot(gi < ngv && w.uhi >= w.ulo && t.any && w.v0 < a.n_v && w.v0 + w.nv > 0);
      if (lane == 0) s_mask = some;
    }
    __syncthreads();
    uint64_t vmask = uniform64(s_mask);
    const bool some = vmask != 0;

    // chunk of columns being worked on, and the one after it
    struct Chunk {
      int view, u, cols, ch, uhi, v0, nv, n, kind;
    };
    auto advance = [&](Chunk& c) -> bool {
      c.u += c.ch;
      if (c.u > c.uhi) {
        if (vmask == 0) return false;
        const int j = __builtin_ctzll(vmask);
        vmask &= vmask - 1;
        c.view = (batch + j) * a.splits + sv0;
        const Window& w = s_win[j];
        c.u = __builtin_amdgcn_readfirstlane(w.ulo);
        c.uhi = __builtin_amdgcn_readfirstlane(w.uhi);
        c.v0 = __builtin_amdgcn_readfirstlane(w.v0);
        c.nv = __builtin_amdgcn_readfirstlane(w.nv);
        c.n = __builtin_amdgcn_readfirstlane(w.n);
        c.kind = __builtin_amdgcn_readfirstlane(w.kind);
        c.ch = min(CH, CAP / (c.nv + kRowPad));
      }
      c.cols = min(c.ch, c.uhi - c.u + 1);
      return true;
    };

    // the chunk's column lines, one per lane (one wavefront)
    auto lines = [&](const Chunk& c, Lines& o) {
      const int lane = here(tid), z0 = here_u(zt);
      const double* v = a.views + 12 * (size_t)c.view;
      const double u = (double)(c.u + lane);
      const Column col = column_line(v, cone, u);
      const double rm = col.m == 0 ? col.r0 : col.r1, ra = col.m == 0 ? col.r1 : col.r0;
      const double d2 = v[5] + u * v[8] + (v[11] < 0.0 ? (double)(a.n_v - 1) * v[11] : 0.0) +
                        (double)c.v0 * fabs(v[11]);
      if (lane < CH) {
        o.sm[lane] = col.m == 0 ? col.s0 : col.s1;
        o.sa[lane] = col.m == 0 ? col.s1 : col.s0;
        o.ga[lane] = ra / rm;
        o.irm[lane] = (col.m == m && lane < c.cols) ? 1.0 / rm : 0.0;
        o.a0[lane] = (cone ? v[2] : d2) - (double)z0;
        o.a1[lane] = cone ? d2 - v[2] : v[2];
      }
      if (lane == 0) o.dv = fabs(v[11]);
    };

    // the chunk's rays to LDS, one wavefront per column, without passing
    // through registers; rows off the detector read as zero (buffer range)
    auto stage = [&](const Chunk& c) {
      const int lane = here(tid);
      const bool flip = (c.kind & kFlip) != 0;
      const int stride = c.nv + kRowPad;
      const int vl = flip ? a.n_v - 1 - c.v0 - lane : c.v0 + lane;
      const int step = flip ? -64 : 64;
      const float* src = a.rays + ((size_t)c.view * a.n_u + c.u) * a.n_v;
      const uint32_t m0 = save_m0();
      for (int k = pl; k < c.cols; k += P) {
        const uint64_t base = (uint64_t)(uintptr_t)(src + (size_t)k * a.n_v);
        const u4rsrc rs = {(uint32_t)base, (uint32_t)(base >> 32) & 0xffffu, (uint32_t)a.n_v * 4u,
                           0x00020000u};
        uint32_t dst = lds_offset(s_buf + k * stride);
        int vi = vl;
        for (int e = 0; e < stride; e += 64, vi += step, dst += 256u)
          if (lane < stride - e) load_to_lds(rs, (uint32_t)vi * 4u, dst);
      }
      restore_m0(m0);
    };

    auto compute = [&](const Chunk& c, const Lines& o) {
      const int lane = here(tid), plane = pm0 + here_u(pl), ra0 = here_u(tr) * R;
      const int stride = c.nv + kRowPad;
      // lane j: column c.u + j on this wavefront's plane
      const int lc = CH < 64 ? min(lane, CH - 1) : lane;
      const double dp = (double)plane - o.sm[lc], irm = o.irm[lc];
      const double pa = o.sa[lc] + dp * o.ga[lc];
      const double t = dp * irm;
      const double B = cone ? t * o.dv : o.dv;
      // from the tile's first row (rows past the grid are not stored)
      const float pr = (float)(pa - (double)ra0);
      bool ok = irm != 0.0 && lane < CH && plane < nm && pr > -1.0f && pr < (float)R;
      if (a.G.clip) {
        const double dx = (m == 0 ? (double)plane : pa) - a.G.cyl[0];
        const double dy = (m == 0 ? pa : (double)plane) - a.G.cyl[1];
        ok = ok && dx * dx + dy * dy < a.G.cyl_r2;
      }
      const float Bf = (float)B, fl = floorf(pr);
      const float d = (float)(pa - (double)(ra0 + (int)fl));
      const int cell = ok ? (int)fl : -2;
      if (lane < CH) {
        float4* o4 = reinterpret_cast<float4*>(slot + lane);
        o4[0] = make_float4((float)(o.a0[lane] + t * o.a1[lane]), Bf, (float)(B - (double)Bf),
                            1.0f / Bf);
        *reinterpret_cast<float2*>(o4 + 1) = make_float2(
            weight_fn<WF>(d),
            __builtin_bit_cast(float, lds_offset(s_buf) + (uint32_t)(lane * stride) * 4u -
                                          4u * 0x4b400000u));
      }
      __builtin_amdgcn_wave_barrier();
      const float dz1 = (float)(lane * ZL - 1);
      float magic = 12582912.0f;  // 1.5 2^23: adding it rounds to an integer
      float cst[ZL + 2];          // small integers in registers (operands that cost no extra cycle)
#pragma unroll
      for (int k = 0; k < ZL + 2; ++k) cst[k] = (float)k;
#pragma unroll
      for (int k = 0; k < ZL + 2; ++k) asm volatile("" : "+v"(cst[k]));
      asm volatile("" : "+v"(magic));

      auto columns = [&](auto n_) {
        constexpr int N = decltype(n_)::value;
#pragma unroll
        for (int f = -1; f < R; ++f) {
          uint64_t mask = __ballot(cell == f);
          while (mask) {
            const int j = __builtin_ctzll(mask);
            mask &= mask - 1;
            const float4 x = *reinterpret_cast<const float4*>(slot + j);
            const float2 y = *reinterpret_cast<const float2*>(&slot[j].w);
            // first candidate: the first ray above z - 1, the ceiling of
            // (z - 1 - A) / B as round(. + 1/2)
            const float tm = __builtin_fmaf(dz1 - x.x, x.w, 0.5f) + magic;
            const float kf = tm - magic;
            const lds_ptr p = (lds_ptr)(uintptr_t)((__builtin_bit_cast(uint32_t, tm) << 2) +
                                                   __builtin_bit_cast(uint32_t, y.y));
            // its distance from z - 1, A + k B - (z - 1): the product and z - 1
            // cancel in one rounding, and B carries its remainder
            float qi = __builtin_fmaf(kf, x.z, __builtin_fmaf(kf, x.y, -dz1) + x.x);
            float s[ZL];
#pragma unroll
            for (int k = 0; k < ZL; ++k) s[k] = 0.0f;
            if constexpr (N > 0) {
              float v[N];
#pragma unroll
              for (int i = 0; i < N; ++i) v[i] = p[i];
#pragma unroll
              for (int i = 0; i < N; ++i) {
#pragma unroll
                for (int k = 0; k < ZL; ++k) {
                  if (i * List<ZL, N>::lo >= k + 2.0 || (i + 1) * List<ZL, N>::hi <= k) continue;
                  float w;
                  if (WF == W_LINEAR && (i + 1) * List<ZL, N>::hi <= k + 1.0)
                    w = sub_clamp(qi, cst[k]);  // below voxel z + k
                  else if (WF == W_LINEAR && i * List<ZL, N>::lo >= k + 1.0)
                    w = sub_clamp(cst[k + 2], qi);  // above it
                  else
                    w = tent<WF>(qi - cst[k + 1]);
                  s[k] = __builtin_fmaf(v[i], w, s[k]);
                }
                qi += x.y;
              }
            } else {
              const lds_ptr end = (lds_ptr)(uintptr_t)(lds_offset(s_buf) + 4u * (CAP - 1));
              for (int i = 0; i < c.n; ++i) {
                const float v = p + i < end ? p[i] : 0.0f;
#pragma unroll
                for (int k = 0; k < ZL; ++k)
                  s[k] = __builtin_fmaf(v, tent<WF>(qi - cst[k + 1]), s[k]);
                qi += x.y;
              }
            }
            const float wb = 1.0f - y.x;
#pragma unroll
            for (int k = 0; k < ZL; ++k) {
              if (f >= 0) acc[f < 0 ? 0 : f][k] = __builtin_fmaf(y.x, s[k], acc[f < 0 ? 0 : f][k]);
              if (f + 1 < R)
                acc[f + 1 < R ? f + 1 : 0][k] =
                    __builtin_fmaf(wb, s[k], acc[f + 1 < R ? f + 1 : 0][k]);
            }
          }
        }
      };
      const int kind = c.kind & ~kFlip;
      auto run = [&](auto n_) {
        if (kind == decltype(n_)::value) columns(n_);
      };
      each_list<ZL>(run);
      if (kind == 0) columns(std::integral_constant<int, 0>());
    };

    Chunk cur = {0, 0, 0, 0, -1, 0, 0, 0, 0};
    bool has = advance(cur);
    int par = 0, turn = 0;
    if (has && pl == 0) lines(cur, s_line[0]);
    for (;;) {
      __syncthreads();  // the previous chunk has been used
      if (!has) break;
      stage(cur);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      Chunk next = cur;
      const bool more = advance(next);
      turn = turn + 1 == P ? 0 : turn + 1;
      if (more && pl == turn) lines(next, s_line[par ^ 1]);
      compute(cur, s_line[par]);
      cur = next;
      has = more;
      par ^= 1;
    }

    // Add the accumulators to the volume (or store them) and clear them:
    // partial sums of at most kViews views keep the rounding error of long sums
    // down. (Nothing to add where no view has rays on the tile: half of a launch whose
    // few views the other axis drives.)
    const int plane = pm0 + pl;
    if (plane < nm && (store || some)) {
      const int z = zt + here(tid) * ZL, ra0 = tr * R;
      const size_t sr = m == 0 ? (size_t)n2 : (size_t)a.G.n[1] * n2;
      const size_t sp = m == 0 ? (size_t)a.G.n[1] * n2 : (size_t)n2;
      float* o = a.vol + (size_t)slice * a.slice + (size_t)plane * sp + (size_t)ra0 * sr + z;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (ra0 + r < na) {
#pragma unroll
          for (int k = 0; k < ZL; ++k)
            if (z + k < n2) o[k] = store ? acc[r][k] : o[k] + acc[r][k];
        }
        o += sr;
      }
    }
    store = false;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int k = 0; k < ZL; ++k) acc[r][k] = 0.0f;
  }
}

// Rays of the sinogram times their step lengths, one wavefront per detector
// column of a view.
__global__ __launch_bounds__(256) void adj_scale_kernel(const GridGeom G,
                                                        const double* __restrict__ views,
                                                        const float* __restrict__ sino, int n_u,
                                                        int n_v, long long n_cols,
                                                        float* __restrict__ out) {
  const long long col = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= n_cols) return;
  const int view = __builtin_amdgcn_readfirstlane((int)(col / n_u));
  const int u = __builtin_amdgcn_readfirstlane((int)(col - (long long)view * n_u));
  const double* v = views + 12 * (size_t)view;
  const bool cone = G.beam == BEAM_CONE;
  const Column c = column_line(v, cone, (double)u);
  const double irm = 1.0 / (c.m == 0 ? c.r0 : c.r1);
  const double wa = (c.m == 0 ? c.r1 : c.r0) * irm * (c.m == 0 ? G.vs[1] : G.vs[0]);
  const double wm = c.m == 0 ? G.vs[0] : G.vs[1];
  const double q = wa * wa + wm * wm;
  const double g0 = (cone ? v[5] + (double)u * v[8] - v[2] : v[2]) * irm * G.vs[2];
  const double gs = cone ? v[11] * irm * G.vs[2] : 0.0;
  const float* src = sino + ((size_t)view * n_u + u) * n_v;
  float* dst = out + ((size_t)view * n_u + u) * n_v;
  for (int e = threadIdx.x & 63; e < n_v; e += 64) {
    const double g = g0 + (double)e * gs;
    dst[e] = src[e] * __builtin_sqrtf((float)(q + g * g));
  }
}

// Sum of n_slices partial volumes, added to vol if accumulate.
__global__ __launch_bounds__(256) void adj_sum_kernel(const float* __restrict__ part, size_t slice,
                                                      int n_slices, int accumulate,
                                                      float* __restrict__ vol) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < slice; i += (size_t)gridDim.x * 256) {
    float s = part[i];
    for (int k = 1; k < n_slices; ++k) s += part[(size_t)k * slice + i];
    vol[i] = accumulate ? vol[i] + s : s;
  }
}

}  // namespace

template <int ZL>
static int run_tiles(const gjp_geometry* g, TileArgs& a, int slices, hipStream_t s) {
  a.nzb = (g->n[2] + 64 * ZL - 1) / (64 * ZL);
  unsigned long long nwg = 0;
  for (int m = 0; m < 2; ++m) {
    if (!a.both && m != a.m0) continue;
    const unsigned long long t = (unsigned long long)((g->n[m] + P - 1) / P) *
                                 ((g->n[1 - m] + R - 1) / R) * a.nzb;
    if (t > nwg) nwg = t;
  }
  if (nwg > 0x7fffffffull) return set_error(-4, "adjoint: volume too large for one launch");
  const dim3 grid((unsigned)nwg, (unsigned)slices);
  if (g->weight == W_SPLINE)
    adj_tile_kernel<W_SPLINE, ZL><<<grid, P * 64, 0, s>>>(a);
  else
    adj_tile_kernel<W_LINEAR, ZL><<<grid, P * 64, 0, s>>>(a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess)
    return set_error(-3, std::string("adjoint tile kernel: ") + hipGetErrorString(e));
  return 0;
}

int launch_adjoint_scale(const gjp_geometry* g, const double* views, const float* sino, int n_views,
                         float* out, hipStream_t s) {
  const long long n_cols = (long long)n_views * g->n_u;
  const long long nb = (n_cols + 3) / 4;
  if (nb > 0x7fffffffll) return set_error(-4, "adjoint: view chunk too large");
  adj_scale_kernel<<<(unsigned)nb, 256, 0, s>>>(g->gg, views, sino, g->n_u, g->n_v, n_cols, out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess)
    return set_error(-3, std::string("adjoint scale kernel: ") + hipGetErrorString(e));
  return 0;
}

int launch_adjoint_tiles(const gjp_geometry* g, const double* views, const float* proj,
                         const float* rays, int n_views, int axes, bool accumulate, float* vol,
                         float* part, int splits, hipStream_t s) {
  TileArgs a;
  a.G = g->gg;
  a.views = views;
  a.proj = proj;
  a.rays = rays;
  a.vol = part ? part : vol;
  a.slice = (size_t)g->n[0] * g->n[1] * g->n[2];
  a.n_views = n_views;
  a.n_u = g->n_u;
  a.n_v = g->n_v;
  a.accumulate = accumulate ? 1 : 0;
  a.splits = 1;
  a.both = 0;
  // two voxels per lane unless one wavefront's 64 cover axis 2 (64 voxels take
  // 0.72 of the time of 128), or the wider tile's window would not fit
  const bool one = g->n[2] <= 64 || g->tile_rows[1] > kTileMaxRows;
  auto run = [&](int slices) { return one ? run_tiles<1>(g, a, slices, s) : run_tiles<2>(g, a, slices, s); };
  const bool both = axes == 3;
  a.m0 = axes == 2 ? 1 : 0;
  if (!part || (!both && splits == 1)) {  // into the volume, one launch per driving axis
    a.vol = vol;
    int st = run(1);
    a.m0 = 1;
    a.accumulate = 1;
    if (st == 0 && both) st = run(1);
    return st;
  }
  a.accumulate = 0;
  a.splits = splits;
  a.both = both ? 1 : 0;
  const int slices = both ? 2 * splits : splits;
  const int st = run(slices);
  if (st != 0) return st;
  return launch_adjoint_sum(part, a.slice, slices, accumulate, vol, s);
}

int launch_adjoint_sum(const float* part, size_t slice, int n_slices, bool accumulate, float* vol,
                       hipStream_t s) {
  const size_t nb = (slice + 255) / 256;
  adj_sum_kernel<<<(unsigned)(nb < 4096 ? nb : 4096), 256, 0, s>>>(part, slice, n_slices,
                                                                  accumulate ? 1 : 0, vol);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_error(-3, std::string("adjoint sum kernel: ") + hipGetErrorString(e));
  return 0;
}

}  // namespace gjp
