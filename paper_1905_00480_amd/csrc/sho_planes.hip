// sho_planes.hip -- the plane form of the projection: one, two or four waves per
// (atom plane, 16 or 32 bands), the x and y passes on FP64 matrix cores, plane
// sums to memory, then one z pass over all atoms.
//
// What bounds the projection is the re-reading of psi: overlapping supports
// read every covered value once per atom (2.3 times at 128^3 / 512 atoms /
// cut-off 5, 18 times at 160^3 / 2048 atoms / cut-offs 3..9).  The item form
// (one workgroup per atom) reads from behind the L2 at 5.6 TB/s.  Here the
// unit of work is an atom plane, and the units are launched plane by plane of
// the grid, one plane per XCD at a time and one band group at a time: a 160^2
// plane of 16 bands is 3.3 MB, so the units resident on an XCD meet in its 4 MB L2
// (measured read rates: 19 TB/s from L2, 7 from the memory-side cache, 6 from
// HBM).  Sixteen bands are also one 128-byte line per grid point.
//
// Lanes: quarter q = lane / 16, band = lane % 16.  v_mfma_f64_4x4x4 (four
// blocks of 4x4x4) computes D[i][j] += A[i][k] B[k][j] per block with A[i][k]
// in lane 16 k + 4 blk + i, B[k][j] in lane 16 k + 4 blk + j and D[i][j] in
// lane 16 i + 4 blk + j: with j = 4 blk + j as the band, B holds 4 rows of 16
// bands and D 4 rows of 16 bands, and A is the same 4x4 matrix in every block.
//   x pass  T1[nx][b]     += phi_nx(x) psi[x][b]      (i = nx, k = x)
//   y pass  T2[nx][ny][b] += phi_ny(y) T1[y][nx][b]   (i = ny, k = y: four runs)
// so no function is padded beyond a multiple of four, no value is reduced
// across lanes, and every sum has a fixed order (no atomics).  The 4x4x4 form
// measured 72 TFLOP/s here, the vector FMA 59 and the 16x16x4 form 48.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sho_device.hpp"
#include "sho_launch.hpp"

namespace sho {
namespace planes {

constexpr uint32_t kOut = 0x80000000u;  // byte offset past every buffer range

__device__ inline double mfma4(double a, double b, double d) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, d, 0, 0, 0);
}

// Buffer descriptor of a range of less than 2^31 bytes: loads outside it
// return zero and touch no memory.
__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}

// NB adjacent values at byte off of the range.  The address unit takes 16
// cycles for 64 lanes of 8 or of 16 bytes alike (it was 85 % busy with 8-byte
// loads), so a lane takes two adjacent bands where there are that many; buffer
// loads need no more than dword alignment.
template <typename T, int NB>
__device__ inline void load_bands(__amdgpu_buffer_rsrc_t r, uint32_t off, double (&v)[NB]) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  typedef unsigned int u4 __attribute__((ext_vector_type(4)));
  if constexpr (sizeof(T) * NB == 16) {
    const u4 x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0);
    v[0] = __builtin_bit_cast(double, u2{x[0], x[1]});
    v[1] = __builtin_bit_cast(double, u2{x[2], x[3]});
  } else if constexpr (sizeof(T) * NB == 8) {
    const u2 x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0);
    if constexpr (NB == 1) {
      v[0] = __builtin_bit_cast(double, x);
    } else {
      v[0] = (double)__builtin_bit_cast(float, (unsigned int)x[0]);
      v[1] = (double)__builtin_bit_cast(float, (unsigned int)x[1]);
    }
  } else {
    v[0] = (double)__builtin_bit_cast(
        float, (unsigned int)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
  }
}

// Exchanges quarters between two registers: swap32 the upper half of a with
// the lower half of b, swap16 the odd quarters of a with the even ones of b.
__device__ inline void swap32(double &a, double &b) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  const u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
  const auto l = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
  a = __builtin_bit_cast(double, u2{l[0], h[0]});
  b = __builtin_bit_cast(double, u2{l[1], h[1]});
}
__device__ inline void swap16(double &a, double &b) {
  typedef unsigned int u2 __attribute__((ext_vector_type(2)));
  const u2 x = __builtin_bit_cast(u2, a), y = __builtin_bit_cast(u2, b);
  const auto l = __builtin_amdgcn_permlane16_swap(x[0], y[0], false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(x[1], y[1], false, false);
  a = __builtin_bit_cast(double, u2{l[0], h[0]});
  b = __builtin_bit_cast(double, u2{l[1], h[1]});
}

// r[k] quarter i <-> r[i] quarter k.
__device__ inline void transpose4(double (&r)[4]) {
  swap32(r[0], r[2]);
  swap32(r[1], r[3]);
  swap16(r[0], r[1]);
  swap16(r[2], r[3]);
}

// Doubles of T2 per lane: groups of four ny for every nx.
constexpr int pair_groups(int nu) {
  int n = 0;
  for (int nx = 0; nx <= nu; ++nx) n += (nu - nx) / 4 + 1;
  return n;
}

// Neighbouring lanes hold the real (even band) and imaginary part of a
// complex band: v <- e^{i th} v with sg = -sin th on real lanes, + on others.
__device__ inline double rotate(double v, double c, double sg) {
  return fma(sg, __shfl_xor(v, 1), c * v);
}

// The waves that share a unit: this one, how many, and this thread's place.
struct Team {
  int w, nw, thread;
};

// Adds up one plane.  Its sums, pair (nx, ny) at ny NF - ny (ny - 1) / 2 + nx, go
// to the plane's place in the plane sums p2, or (kLds) to p2 in LDS, 16 bands per
// pair.  NB: adjacent bands per lane (16 NB per wave).  The barriers are the
// workgroup's: one, with several waves to a team three, also for a unit without
// bundles.
template <typename T, int NU, int NB, bool kLds>
__device__ inline void project_plane(const PlaneArgs &P, const PlaneUnit &U, int group,
                                     const T *__restrict__ psi, T *__restrict__ p2, char *lds,
                                     const Team &team) {
  constexpr int NF = NU + 1;
  constexpr int NG = pair_groups(NU);
  constexpr int S = (NF + 3) / 4;  // groups of four functions
  constexpr int W = 4 * S;         // table row in LDS
  constexpr bool kDeep = NB == 1 || NU <= 7;
  const int lane = threadIdx.x & 63;
  const int w = team.w, nw = team.nw;
  const int q = lane >> 4, i4 = lane & 3;
  const int band = (group * 16 + (lane & 15)) * NB;
  const int nfp = U.nfp;
  const uint32_t bytes_x = (uint32_t)P.B * (uint32_t)sizeof(T);
  const int nb = U.nb;
  // LDS: the unit's bundles, and the atom's x rows of W functions (to a
  // multiple of four points, zeros past the last)
  PlaneBundle *bun = reinterpret_cast<PlaneBundle *>(lds);
  double *tab = reinterpret_cast<double *>(lds + P.lds_bundles * sizeof(PlaneBundle));
  const double *gx = P.tab + U.tab_off;
  const double *gy = gx + (int64_t)U.mx * nfp + i4;
  {
    const int nt = ((U.mx + 3) & ~3) * W;
    const int4 *src = reinterpret_cast<const int4 *>(P.bundles + U.b0);
    constexpr int K = 6;  // loads in flight per lane
    const int threads = nw * 64;
    for (int t0 = team.thread; t0 < max(nt, 3 * nb); t0 += K * threads) {
      double v[K];
      int4 c = make_int4(0, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < K; ++u) {
        const int t = t0 + u * threads, x = t / W, n = t % W;
        v[u] = x < U.mx ? gx[x * nfp + n] : 0.0;
      }
      if (t0 < 3 * nb) c = src[t0];
#pragma unroll
      for (int u = 0; u < K; ++u)
        if (t0 + u * threads < nt) tab[t0 + u * threads] = v[u];
      if (t0 < 3 * nb) reinterpret_cast<int4 *>(bun)[t0] = c;
#pragma unroll
      for (int u = 1; u < K; ++u) {
        const int t = t0 + u * threads;
        if (t < 3 * nb) reinterpret_cast<int4 *>(bun)[t] = src[t];
      }
    }
  }
  __syncthreads();
  // the buffer starts mx points before the memory plane, so that no offset is
  // negative; lanes with a band read only points of the unit's runs (the
  // others what follows there, into sums that are not stored)
  const __amdgpu_buffer_rsrc_t rsrc =
      buffer_of(psi + ((int64_t)U.z * P.ny * P.nx - U.mx) * P.B,
                ((uint32_t)P.ny * P.nx + U.mx) * bytes_x);
  double T2[NB][NG];  // [nx][ny group]: quarter = ny mod 4
  double T1[NB][4][S];
#pragma unroll
  for (int h = 0; h < NB; ++h) {
#pragma unroll
    for (int k = 0; k < NG; ++k) T2[h][k] = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int s = 0; s < S; ++s) T1[h][r][s] = 0.0;
  }
  // the lane's byte offset at x step 0
  const uint32_t vl = (uint32_t)q * bytes_x + (uint32_t)band * (uint32_t)sizeof(T);
  // the bundle whose loads are being issued
  uint32_t off[4];
  int jx0[4], len[4];
  double fy[S];  // y rows of the bundle that is being contracted (run q)
  int b = w, t = 0, t1 = 0, i0 = 0, i1 = 0;
  auto open_bundle = [&](int bb) {
    const PlaneBundle *p = bun + bb;
    const uint4 o = *reinterpret_cast<const uint4 *>(p->off);
    const uint4 x = *reinterpret_cast<const uint4 *>(p->jx0);
    const uint2 st = *reinterpret_cast<const uint2 *>(&p->t0);
    off[0] = o.x, off[1] = o.y, off[2] = o.z, off[3] = o.w;
    jx0[0] = x.x & 0xffff, jx0[1] = x.x >> 16, jx0[2] = x.y & 0xffff, jx0[3] = x.y >> 16;
    len[0] = x.z & 0xffff, len[1] = x.z >> 16, len[2] = x.w & 0xffff, len[3] = x.w >> 16;
    const uint32_t a = __builtin_amdgcn_readfirstlane(st.x);
    const uint32_t c = __builtin_amdgcn_readfirstlane(st.y);
    t = (int)(a & 0xffff);
    t1 = (int)(a >> 16);
    i0 = (int)(c & 0xffff);
    i1 = (int)(c >> 16);
  };
  auto load_fy = [&](int bb) {
    const double *f = gy + (int)bun[bb].jy[q] * nfp;
#pragma unroll
    for (int g = 0; g < S; ++g) fy[g] = f[4 * g];
  };
  // Loads of step t: the offsets need masks only where a run begins or ends;
  // the loads themselves are issued on one path, so that the compiler's waits
  // count them (past the last step every lane is masked: no memory is touched).
  auto issue = [&](double (&v)[4][NB]) {
    const uint32_t vo = (uint32_t)(4 * t) * bytes_x + vl;
    uint32_t o[4];
    if (t >= i0 && t < i1) {
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = vo + off[r];
    } else {
      const int x = 4 * t + q;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool ok = (uint32_t)(x - jx0[r]) < (uint32_t)len[r];
        o[r] = ok ? vo + off[r] : kOut;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) load_bands<T, NB>(rsrc, o[r], v[r]);
  };
  auto contract = [&](const double (&cur)[4][NB], int tc) {
    const double *f = tab + (4 * tc + q) * W + i4;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const double a = f[4 * s];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int h = 0; h < NB; ++h) T1[h][r][s] = mfma4(a, cur[r][h], T1[h][r][s]);
    }
  };
  // y pass of bundle bb: four runs at once
  auto ypass = [&](int bb) {
    if (P.phase) {
      // the runs of a bundle lie in one periodic image, which carries
      // e^{+i k.T}
      const cptr<double> cs = as_const(P.phase) + 2 * (U.b0 + bb);
      const double c = cs[0], sn = cs[1];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int s = 0; s < S; ++s) {
          if constexpr (NB == 2) {  // the lane holds both parts
            const double re = T1[0][r][s], im = T1[1][r][s];
            T1[0][r][s] = fma(-sn, im, c * re);
            T1[1][r][s] = fma(sn, re, c * im);
          } else {
            T1[0][r][s] = rotate(T1[0][r][s], c, (lane & 1) ? sn : -sn);
          }
        }
    }
#pragma unroll
    for (int h = 0; h < NB; ++h) {
      int k = 0;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        double o[4] = {T1[h][0][s], T1[h][1][s], T1[h][2][s], T1[h][3][s]};
        transpose4(o);  // o[i]: function 4 s + i, quarter = run
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int nx = 4 * s + i;
          if (nx > NU) continue;
#pragma unroll
          for (int g = 0; 4 * g <= NU - nx; ++g, ++k) T2[h][k] = mfma4(fy[g], o[i], T2[h][k]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) T1[h][r][s] = 0.0;
      }
    }
  };
  // Three register buffers: two steps are in flight while a third is
  // contracted, across the bundles of the wave too (two buffers where the
  // sums leave no registers for three).  A buffer remembers its
  // table step and whether it ends its bundle (1) or the wave's work (3).
  // After the last step buffers are filled with zeros (every lane masked) and
  // contracted into sums that nothing reads: a round of three steps has no
  // exit inside, which would make the waits at its top count the loads of the
  // abandoned path.  The y rows of the next bundle are requested behind its
  // first steps.
  struct Step {
    int t, end;
  };
  int bo = w;  // the bundle whose loads are being issued
  bool done = false;
  auto next = [&](double (&v)[4][NB], Step &d) {
    issue(v);
    d.t = min(t, t1 - 1);
    d.end = 0;
    if (bo < nb && ++t >= t1) {
      bo += nw;
      d.end = bo < nb ? 1 : 3;
      if (bo < nb) open_bundle(bo);
    }
  };
  auto step = [&](const double (&cur)[4][NB], const Step &d, double (&nxt)[4][NB], Step &dn) {
    next(nxt, dn);
    contract(cur, d.t);
    if (d.end) {
      ypass(b);
      b += nw;
      if (d.end == 1)
        load_fy(b);
      else
        done = true;
    }
  };
  if (b < nb) {
    open_bundle(b);
    load_fy(b);
    double v0[4][NB], v1[4][NB];
    Step d0, d1;
    next(v0, d0);
    if constexpr (kDeep) {
      double v2[4][NB];
      Step d2;
      next(v1, d1);
      do {
        step(v0, d0, v2, d2);
        step(v1, d1, v0, d0);
        step(v2, d2, v1, d1);
      } while (!done);
    } else {
      do {
        step(v0, d0, v1, d1);
        step(v1, d1, v0, d0);
      } while (!done);
    }
  }
  // the waves' sums meet in LDS (over the tables) and are added in wave
  // order, every wave taking its share of the pair groups
  double *red = reinterpret_cast<double *>(lds);
  if (nw > 1) {
    __syncthreads();
#pragma unroll
    for (int h = 0; h < NB; ++h)
#pragma unroll
      for (int k = 0; k < NG; ++k) red[((w * NB + h) * NG + k) * 64 + lane] = T2[h][k];
    __syncthreads();
  }
  T *dst = p2 + (kLds ? (int64_t)(lane & 15) : U.sums * P.B + band);
  const bool pairs = !kLds && NB == 2 && (P.B & 1) == 0;  // (the scratch is aligned)
  int k = 0;
#pragma unroll
  for (int nx = 0; nx < NF; ++nx) {
#pragma unroll
    for (int g = 0; 4 * g <= NU - nx; ++g, ++k) {
      if ((k & (nw - 1)) != w) continue;
      double sum[NB];
#pragma unroll
      for (int h = 0; h < NB; ++h) {
        sum[h] = T2[h][k];
        if (nw > 1) {
          sum[h] = red[(h * NG + k) * 64 + lane];
          for (int i = 1; i < nw; ++i) sum[h] += red[((i * NB + h) * NG + k) * 64 + lane];
        }
      }
      const int ny = 4 * g + q;
      const int pair = ny * NF - ny * (ny - 1) / 2 + nx;
      T *o = dst + (kLds ? (int64_t)16 * pair : (int64_t)pair * P.B);
      if (ny > NU - nx) continue;
      if constexpr (kLds) {
        *o = (T)sum[0];
        continue;
      }
      if constexpr (NB == 2) {
        if (pairs && band < P.B) {
          struct __attribute__((aligned(2 * sizeof(T)))) T2v {
            T a, b;
          };
          *reinterpret_cast<T2v *>(o) = T2v{(T)sum[0], (T)sum[1]};
        }
      }
      if (!pairs) {
#pragma unroll
        for (int h = 0; h < NB; ++h)
          if (band + h < P.B) o[h] = (T)sum[h];
      }
    }
  }
}

#define SHO_NU_CASES(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)

// waves per SIMD the register allocator must allow
constexpr int waves(int numax, int nb) {
  return nb == 1 ? (numax <= 7 ? 4 : numax <= 9 ? 3 : 2) : (numax <= 3 ? 4 : 2);
}

template <typename T, int NUMAX, int NB>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(waves(NUMAX, NB)))) void k_project_planes(
    PlaneArgs P, const T *__restrict__ psi, T *__restrict__ p2) {
  extern __shared__ double lds[];
  const PlaneUnit U = load_uniform(P.units + blockIdx.x);
  if (U.nu < 0) return;  // padding of the XCD-dealt launch
  const Team team{wave_id(), (int)blockDim.x >> 6, (int)threadIdx.x};
  switch (U.nu) {
#define X(N)                                                                                  \
  case N:                                                                                     \
    if constexpr (N <= NUMAX)                                                                 \
      project_plane<T, N, NB, false>(P, U, blockIdx.y, psi, p2, (char *)lds, team);           \
    break;
    SHO_NU_CASES(X)
#undef X
  }
}

// z pass: c[n][b] = h^3 sum_jz phi_nz(z_jz) P2[jz][nx,ny][b] for all atoms in
// one launch; thread = (pair, NB adjacent bands), every plane sum read once, kZ
// planes in flight.  Bound by the read of the plane sums.
constexpr int kZThreads = 128;
constexpr int kZ = 4;

template <typename T, int NB>
struct __attribute__((aligned(NB * sizeof(T)))) Bands {
  T v[NB];
};

template <typename T, int NU, int NB>
__device__ inline void zpass_atom(const PlaneArgs &P, int a, const AtomRec &A,
                                  const T *__restrict__ p2, T *__restrict__ c) {
  constexpr int NF = NU + 1;
  constexpr int NP = NF * (NF + 1) / 2;
  const int item = (int)blockIdx.y * kZThreads + (int)threadIdx.x;
  const int p = item >> 4;
  const int b = ((int)blockIdx.z * 16 + (item & 15)) * NB;
  if (p >= NP || b >= P.B) return;
  const cptr<double> tz = as_const(P.tab) + A.tab_off + (int64_t)(A.mx + A.my) * A.tab_nfp;
  int ny = 0, nx = p;  // pair p -> (nx, ny), ny outer
  while (nx >= NF - ny) {
    nx -= NF - ny;
    ++ny;
  }
  const int64_t plane = (int64_t)NP * P.B;
  const T *s = p2 + P.u2_off[a] * P.u2_scale + (int64_t)p * P.B + b;
  double acc[NF][NB];
#pragma unroll
  for (int n = 0; n < NF; ++n)
#pragma unroll
    for (int h = 0; h < NB; ++h) acc[n][h] = 0.0;
  for (int j0 = 0; j0 < A.mz; j0 += kZ) {
    Bands<T, NB> v[kZ];
#pragma unroll
    for (int u = 0; u < kZ; ++u)
      v[u] = *reinterpret_cast<const Bands<T, NB> *>(s + min(j0 + u, A.mz - 1) * plane);
#pragma unroll
    for (int u = 0; u < kZ; ++u) {
      const cptr<double> f = tz + min(j0 + u, A.mz - 1) * A.tab_nfp;
#pragma unroll
      for (int h = 0; h < NB; ++h) {
        const double x = j0 + u < A.mz ? (double)v[u].v[h] : 0.0;
#pragma unroll
        for (int n = 0; n < NF; ++n) acc[n][h] = fma(f[n], x, acc[n][h]);
      }
    }
  }
  // row of (nx, ny, nz): nz-major, then ny, nx fastest
  T *out = c + A.coeff_row * P.B + b;
#pragma unroll
  for (int nz = 0; nz < NF; ++nz) {
    if (nx + ny + nz <= NU) {
      int base = 0;
#pragma unroll
      for (int k = 0; k < nz; ++k) base += (NU - k + 1) * (NU - k + 2) / 2;
      const int m = NU - nz + 1;  // functions nx of row ny = 0 in this layer
      Bands<T, NB> o;
#pragma unroll
      for (int h = 0; h < NB; ++h) o.v[h] = (T)(P.h3 * acc[nz][h]);
      *reinterpret_cast<Bands<T, NB> *>(
          out + (int64_t)(base + ny * m - ny * (ny - 1) / 2 + nx) * P.B) = o;
    }
  }
}

template <typename T, int NUMAX, int NB>
__global__ __launch_bounds__(kZThreads) void k_zpass_all(PlaneArgs P, const T *__restrict__ p2,
                                                         T *__restrict__ c) {
  const int a = P.nu_atoms[blockIdx.x];
  const AtomRec A = load_uniform(P.atoms + a);
  switch (A.nu) {
#define X(N)                                                        \
  case N:                                                           \
    if constexpr (N <= NUMAX) zpass_atom<T, N, NB>(P, a, A, p2, c); \
    break;
    SHO_NU_CASES(X)
#undef X
  }
}

// The same sums without scratch, to the last bit: one workgroup per (atom, 16
// bands), whose teams (the waves of a unit each) take the atom's planes in turn;
// their sums meet in LDS and are added to the coefficients there in the order of
// k_zpass_all.  For deterministic plans where the plane sums may not be used or
// had, so that a call gives the same bits there.  Bound by the latency of a
// team's planes: 128^3, 512 atoms, cut-off 5, 32 bands 329 us (work items of the
// mode 336, plane sums in memory 190); 64^3, 120 atoms, cut-off 9, 64 bands 648
// (2770, 395); 8 uneven atoms, 20 bands 121 (132, 20); 96^3, 300 atoms, cut-off 3,
// 20 bands 141 (118, 53).
struct AtomLds {
  int team, sums, coeff;  // bytes of a team's part, begin of the others
};

template <int NU>
__device__ inline void project_atom(const PlaneArgs &P, const AtomRec &A, const AtomLds &at,
                                    const double *__restrict__ psi, double *__restrict__ c,
                                    char *lds) {
  constexpr int NF = NU + 1;
  constexpr int NS = NF * (NF + 1) * (NF + 2) / 6;
  constexpr int NP = NF * (NF + 1) / 2;
  const int nw = P.waves, own = wave_id() / nw, teams = (int)blockDim.x / (64 * nw);
  const Team team{wave_id() % nw, nw, (int)threadIdx.x - own * nw * 64};
  double *sums = reinterpret_cast<double *>(lds + at.sums);  // [team][pair][16 bands]
  double *acc = reinterpret_cast<double *>(lds + at.coeff);  // [row][16 bands]
  const cptr<double> tz = as_const(P.tab) + A.tab_off + (int64_t)(A.mx + A.my) * A.tab_nfp;
  // every coefficient is one thread's: item = (pair, band), all nz
  auto rows = [&](int item, auto &&f) {  // f(nz, coefficient row) of the pair
    const int p = item >> 4;
    int ny = 0, nx = p;  // pair p -> (nx, ny), ny outer
    while (nx >= NF - ny) {
      nx -= NF - ny;
      ++ny;
    }
    int base = 0;  // row of (nx, ny, nz): nz-major, then ny, nx fastest
#pragma unroll 1
    for (int nz = 0; nz <= NU - nx - ny; ++nz) {
      const int m = NF - nz;  // functions nx of row ny = 0 in this layer
      f(nz, base + ny * m - ny * (ny - 1) / 2 + nx);
      base += m * (m + 1) / 2;
    }
  };
  for (int t = threadIdx.x; t < NS * 16; t += blockDim.x) acc[t] = 0.0;
  for (int j0 = 0; j0 < A.mz; j0 += teams) {
    PlaneUnit U{};  // (no bundles: past the last plane)
    if (j0 + own < A.mz) U = load_uniform(P.units + P.plane_unit[A.plane_begin + j0 + own]);
    project_plane<double, NU, 1, true>(P, U, blockIdx.y, psi,
                                       sums + own * NP * 16, lds + own * at.team, team);
    __syncthreads();
    const int n = min(teams, A.mz - j0);
    for (int t = threadIdx.x; t < NP * 16; t += blockDim.x)
      rows(t, [&](int nz, int row) {
        double &a = acc[row * 16 + (t & 15)];
        double v = a;
        for (int i = 0; i < n; ++i)
          v = fma(tz[(j0 + i) * A.tab_nfp + nz], sums[i * NP * 16 + t], v);
        a = v;
      });
  }
  for (int t = threadIdx.x; t < NP * 16; t += blockDim.x)
    rows(t, [&](int nz, int row) {
      const int band = (int)blockIdx.y * 16 + (t & 15);
      double v = acc[row * 16 + (t & 15)];
      // (the z pass fills its last round of planes up with zeros, which may turn
      // the sign of a zero)
      if (A.mz % kZ) v = fma(tz[(A.mz - 1) * A.tab_nfp + nz], 0.0, v);
      if (band < P.B) c[(A.coeff_row + row) * P.B + band] = P.h3 * v;
    });
}

constexpr int atom_threads(int numax) { return numax <= 7 ? 1024 : 512; }  // (registers)

template <int NUMAX>
__global__ __launch_bounds__(atom_threads(NUMAX)) void k_project_atoms(
    PlaneArgs P, AtomLds at, const double *__restrict__ psi, double *__restrict__ c) {
  extern __shared__ double lds[];
  const AtomRec A = load_uniform(P.atoms + P.nu_atoms[blockIdx.x]);
  switch (A.nu) {
#define X(N)                                                                   \
  case N:                                                                      \
    if constexpr (N <= NUMAX) project_atom<N>(P, A, at, psi, c, (char *)lds); \
    break;
    SHO_NU_CASES(X)
#undef X
  }
}

// LDS of a unit: tables and bundles, then (over them) its waves' sums.
template <int NUMAX>
static size_t unit_lds(const PlaneArgs &P, int nb) {
  constexpr int W = (NUMAX + 4) / 4 * 4;
  return std::max(
      (size_t)P.lds_rows * W * sizeof(double) + (size_t)P.lds_bundles * sizeof(PlaneBundle),
      P.waves > 1 ? (size_t)P.waves * nb * pair_groups(NUMAX) * 64 * sizeof(double) : 0);
}

template <typename T, int NUMAX>
static hipError_t launch_any(const PlaneArgs &P, const void *psi, void *p2, void *c,
                             hipStream_t s) {
  const dim3 g((unsigned)P.nunits, (unsigned)((P.B + 16 * P.nb - 1) / (16 * P.nb)));
  const size_t shm = unit_lds<NUMAX>(P, P.nb);
  if (P.nb == 1)
    hipLaunchKernelGGL((k_project_planes<T, NUMAX, 1>), g, dim3(64u * P.waves), shm, s, P,
                       static_cast<const T *>(psi), static_cast<T *>(p2));
  else
    hipLaunchKernelGGL((k_project_planes<T, NUMAX, 2>), g, dim3(64u * P.waves), shm, s, P,
                       static_cast<const T *>(psi), static_cast<T *>(p2));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // two bands per thread where every pair of bands is whole and aligned
  const bool two = P.B % 2 == 0 && ((uintptr_t)p2 | (uintptr_t)c) % (2 * sizeof(T)) == 0;
  const int per = two ? 32 : 16;
  const dim3 gz((unsigned)P.natoms_u2,
                (unsigned)(((NUMAX + 1) * (NUMAX + 2) / 2 * 16 + kZThreads - 1) / kZThreads),
                (unsigned)((P.B + per - 1) / per));
  if (two)
    hipLaunchKernelGGL((k_zpass_all<T, NUMAX, 2>), gz, dim3(kZThreads), 0, s, P,
                       static_cast<const T *>(p2), static_cast<T *>(c));
  else
    hipLaunchKernelGGL((k_zpass_all<T, NUMAX, 1>), gz, dim3(kZThreads), 0, s, P,
                       static_cast<const T *>(p2), static_cast<T *>(c));
  return hipGetLastError();
}

template <typename T>
static hipError_t launch_t(int nu_max, const PlaneArgs &P, const void *psi, void *p2, void *c,
                           hipStream_t s) {
  if (nu_max <= 3) return launch_any<T, 3>(P, psi, p2, c, s);
  if (nu_max <= 5) return launch_any<T, 5>(P, psi, p2, c, s);
  if (nu_max <= 7) return launch_any<T, 7>(P, psi, p2, c, s);
  if (nu_max <= 9) return launch_any<T, 9>(P, psi, p2, c, s);
  return launch_any<T, 10>(P, psi, p2, c, s);
}

template <int NUMAX>
static hipError_t launch_atoms(const PlaneArgs &P, const double *psi, double *c, hipStream_t s) {
  constexpr size_t kLds = 160 * 1024;
  const size_t pairs = (NUMAX + 1) * (NUMAX + 2) / 2, row = 16 * sizeof(double);
  const size_t coeff = pairs * (NUMAX + 3) / 3 * row, team = unit_lds<NUMAX>(P, 1);
  // as many teams as fit (one does: at most 42 + 8.3 + 35.8 KB at cut-off 10)
  const int teams = (int)std::min<size_t>(atom_threads(NUMAX) / (64 * P.waves),
                                          (kLds - coeff) / (team + pairs * row));
  if (teams < 1) return hipErrorInvalidValue;
  const AtomLds at{(int)team, (int)(teams * team), (int)(teams * (team + pairs * row))};
  hipLaunchKernelGGL((k_project_atoms<NUMAX>), dim3((unsigned)P.natoms_u2, (unsigned)(P.B + 15) / 16),
                     dim3(64u * P.waves * teams), at.coeff + coeff, s, P, at, psi, c);
  return hipGetLastError();
}

}  // namespace planes

hipError_t launch_project_atoms(int nu_max, const PlaneArgs &P, const double *psi, double *c,
                                hipStream_t s) {
  if (P.natoms_u2 <= 0) return hipSuccess;
  if (!P.plane_unit) return hipErrorInvalidValue;
  if (nu_max <= 3) return planes::launch_atoms<3>(P, psi, c, s);
  if (nu_max <= 5) return planes::launch_atoms<5>(P, psi, c, s);
  if (nu_max <= 7) return planes::launch_atoms<7>(P, psi, c, s);
  if (nu_max <= 9) return planes::launch_atoms<9>(P, psi, c, s);
  return planes::launch_atoms<10>(P, psi, c, s);
}

hipError_t launch_project_planes(int nu_max, bool f32, const PlaneArgs &P, const void *psi,
                                 void *p2, void *c, hipStream_t s) {
  if (P.nunits <= 0) return hipSuccess;
  return f32 ? planes::launch_t<float>(nu_max, P, psi, p2, c, s)
             : planes::launch_t<double>(nu_max, P, psi, p2, c, s);
}

}  // namespace sho
