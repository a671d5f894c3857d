// sho_tiles.hip -- the tile form of the expansion: plane partials, then one
// workgroup per tile of 16 rows x 16 points of one memory plane and 16 or 32
// bands.  Wave w keeps the sums of rows 4 w .. 4 w + 3 (a row per quarter of
// the wave, a band or two per lane) in registers and adds every atom plane:
//   y pass  U[nx][y][b] = sum_ny phi_ny(y) U2[nx][ny][b]
//           by v_mfma_f64_4x4x4 (lane layout in sho_planes.hip; i = y, k = ny),
//           whose result has the row in the quarter that keeps it;
//   x pass  psi[y][x][b] += sum_nx phi_nx(x) U[nx][y][b]
//           by vector FMAs that read phi across the 16 lanes of a quarter.
// Matrix instructions along x were tried first: they pad nx to fours, need U
// transposed and the table values masked per row, and a matrix and a vector
// instruction do not overlap on the FP64 unit (16 cycles a matrix one, 7 the
// first vector one behind it, 3 each further).  At 160^3, 2048 atoms, cut-offs
// 3..9, 64 bands that took 4.62 ms, this 4.22 ms, and tiles of 16 instead of 32
// points (half the registers, four waves per SIMD instead of two, so that one
// workgroup's loads and stores run under another's sums) 3.57 ms.
//
// The block form, which was the default, adds each run point by point through
// LDS atomics: 5.4 ms there; at 64^3, 11 projections per point, cut-off 4, 1024
// bands 2.76 ms against 1.97 here.  psi is read and written once, there are no
// atomics, and the entries of a tile come in a fixed order, so deterministic
// plans take this form too.  An atom plane's partials and table rows are copied
// into LDS by the whole workgroup (direct loads into LDS) ahead of their use.
// Few entries per tile: bound by HBM (128^3, 512 atoms, cut-off 5, 32 bands: 1.12
// GB by counters in 0.20 ms, the rate of a copy).  Many (160^3 and 64^3 above): by
// the latency of each wave's entries, one after the other, with vector
// instructions issued in 44-48 % of the cycles, matrix ones in 12-16 %.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sho_device.hpp"
#include "sho_launch.hpp"

namespace sho {
namespace tiles {

#define SHO_NU_CASES(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)

constexpr int kThreads = 256;
constexpr uint32_t kOut = 0x80000000u;  // byte offset past every buffer range

__device__ inline double mfma4(double a, double b, double d) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, d, 0, 0, 0);
}

__device__ inline __amdgpu_buffer_rsrc_t buffer_of(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00027000);
}

typedef unsigned int u2v __attribute__((ext_vector_type(2)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));

// NB adjacent values at byte off of the range (zeros outside it).
template <typename T, int NB, int kNt>
__device__ inline void load_bands(__amdgpu_buffer_rsrc_t r, uint32_t off, double (&v)[NB]) {
  if constexpr (sizeof(T) * NB == 16) {
    const u4v x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kNt);
    v[0] = __builtin_bit_cast(double, u2v{x[0], x[1]});
    v[1] = __builtin_bit_cast(double, u2v{x[2], x[3]});
  } else if constexpr (sizeof(T) * NB == 8) {
    const u2v x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, kNt);
    if constexpr (NB == 1) {
      v[0] = __builtin_bit_cast(double, x);
    } else {
      v[0] = (double)__builtin_bit_cast(float, (unsigned int)x[0]);
      v[1] = (double)__builtin_bit_cast(float, (unsigned int)x[1]);
    }
  } else {
    v[0] = (double)__builtin_bit_cast(
        float, (unsigned int)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, kNt));
  }
}

// Stores NB adjacent values (nothing outside the range).
template <typename T, int NB, int kNt>
__device__ inline void store_bands(__amdgpu_buffer_rsrc_t r, uint32_t off, const double *v) {
  if constexpr (sizeof(T) == 8) {
    const u2v a = __builtin_bit_cast(u2v, v[0]);
    if constexpr (NB == 2) {
      const u2v b = __builtin_bit_cast(u2v, v[1]);
      __builtin_amdgcn_raw_buffer_store_b128(u4v{a[0], a[1], b[0], b[1]}, r, (int)off, 0, kNt);
    } else {
      __builtin_amdgcn_raw_buffer_store_b64(a, r, (int)off, 0, kNt);
    }
  } else {
    const unsigned int a = __builtin_bit_cast(unsigned int, (float)v[0]);
    if constexpr (NB == 2) {
      const unsigned int b = __builtin_bit_cast(unsigned int, (float)v[1]);
      __builtin_amdgcn_raw_buffer_store_b64(u2v{a, b}, r, (int)off, 0, kNt);
    } else {
      __builtin_amdgcn_raw_buffer_store_b32(a, r, (int)off, 0, kNt);
    }
  }
}

// ---------------------------------------------------------- plane partials --

// U2[jz][p][b] = alpha sum_nz phi_nz(z_jz) C[nx,ny,nz][b] for every plane jz of
// every atom, pairs p with nx outer and ny inner (the order in which the tile
// kernel's lanes read four ny of one nx), for all cut-offs in one launch.
// One workgroup per (atom, 16 NB bands, part of the planes): the coefficients
// in LDS, a thread writes all pairs of one plane and NB bands.  Bound by the
// write.
template <typename T, int NB>
struct __attribute__((aligned(NB * sizeof(T)))) Bands {
  T v[NB];
};

template <typename T, int NU, int NB>
__device__ inline void partials_atom(const TileArgs &E, int a, const AtomRec &A,
                                     const T *__restrict__ c, T *__restrict__ u2,
                                     Bands<T, NB> *cs) {
  constexpr int NF = NU + 1;
  constexpr int NS = NF * (NF + 1) * (NF + 2) / 6;
  constexpr int NP = NF * (NF + 1) / 2;
  const int b0 = (int)blockIdx.y * 16 * NB;
  for (int t0 = threadIdx.x; t0 < NS * 16; t0 += 4 * kThreads) {
    Bands<T, NB> v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = t0 + u * kThreads, n = min(t >> 4, NS - 1);
      const int b = min(b0 + (t & 15) * NB, E.B - NB);  // (a copy past the last)
      v[u] = *reinterpret_cast<const Bands<T, NB> *>(c + (A.coeff_row + n) * E.B + b);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (t0 + u * kThreads < NS * 16) cs[t0 + u * kThreads] = v[u];
  }
  __syncthreads();
  const double *tz = E.tab + A.tab_off + (int64_t)(A.mx + A.my) * A.tab_nfp;
  T *dst = u2 + E.u2_off[a] * E.u2_scale;
  for (int t = threadIdx.x + blockIdx.z * kThreads; t < A.mz * 16; t += gridDim.z * kThreads) {
    const int bl = t & 15, jz = t >> 4;
    const int b = b0 + bl * NB;
    if (b >= E.B) continue;
    double fz[NF];
#pragma unroll
    for (int n = 0; n < NF; ++n) fz[n] = E.alpha * tz[(int64_t)jz * A.tab_nfp + n];
    T *out = dst + (int64_t)jz * NP * E.B + b;
    int p = 0;
#pragma unroll
    for (int nx = 0; nx < NF; ++nx) {
#pragma unroll
      for (int ny = 0; ny < NF - nx; ++ny, ++p) {
        double acc[NB] = {};
#pragma unroll
        for (int nz = 0; nz < NF; ++nz) {
          if (nx + ny + nz > NU) continue;
          int row = nx;  // of (nx, ny, nz): nz-major, then ny, nx fastest
#pragma unroll
          for (int k = 0; k < nz; ++k) row += (NU - k + 1) * (NU - k + 2) / 2;
#pragma unroll
          for (int j = 0; j < ny; ++j) row += NU - nz - j + 1;
          const Bands<T, NB> x = cs[row * 16 + bl];
#pragma unroll
          for (int h = 0; h < NB; ++h) acc[h] = fma(fz[nz], (double)x.v[h], acc[h]);
        }
        Bands<T, NB> o;
#pragma unroll
        for (int h = 0; h < NB; ++h) o.v[h] = (T)acc[h];
        *reinterpret_cast<Bands<T, NB> *>(out + (int64_t)p * E.B) = o;
      }
    }
  }
}

template <typename T, int NUMAX, int NB>
__global__ __launch_bounds__(kThreads) void k_partials(TileArgs E, const T *__restrict__ c,
                                                       T *__restrict__ u2) {
  extern __shared__ char lds[];
  const int a = E.nu_atoms[blockIdx.x];
  const AtomRec A = load_uniform(E.atoms + a);
  switch (A.nu) {
#define X(N)                                                                    \
  case N:                                                                       \
    if constexpr (N <= NUMAX)                                                   \
      partials_atom<T, N, NB>(E, a, A, c, u2, reinterpret_cast<Bands<T, NB> *>(lds)); \
    break;
    SHO_NU_CASES(X)
#undef X
  }
}

// ------------------------------------------------------------------- tiles --

// LDS of one staged entry: the table rows, then the partials [pair][16 NB].
constexpr int kXRows = kTileX, kYRows = kTileRows;
template <typename T, int NB>
constexpr int slot_bytes(int numax) {
  return (kXRows + kYRows) * table_nfp_c(numax) * 8 +
         (numax + 1) * (numax + 2) / 2 * 16 * NB * (int)sizeof(T);
}

// One direct load into LDS: lane i's BYTES from src + off to dst + BYTES i
// (src and the LDS address dst the same in all lanes).  Written out because the builtin makes
// the compiler wait for it before any later LDS read, also of the other slots:
// the copies of the next entries would not overlap this one.  The load has no
// register to write; the kernel waits for vmcnt(0) and a barrier before the
// slot is read.
// (The compiler says of every copy that m0 is a register it keeps for itself; it
// writes m0 in front of each instruction that reads it, and none else does here.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int BYTES>
__device__ inline void to_lds(const char *src, uint32_t off, uint32_t dst) {
  if constexpr (BYTES == 16)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst),
                 "v"(off), "s"(src)
                 : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(dst),
                 "v"(off), "s"(src)
                 : "memory", "m0");
}

#pragma clang diagnostic pop

// A lane's place in the copies of partials: its byte offset from the first
// pair of a 64-lane chunk, and that pair's number in the chunk.
template <typename T, int NB>
struct Place {
  static constexpr int kRow = 16 * NB * (int)sizeof(T);  // bytes of a pair's bands
  static constexpr int kWidePer = kRow / 16;             // lanes per pair, 16 bytes each
  static constexpr int kThinPer = kRow / 4;              // 4 bytes each
  uint32_t off, pair;
  __device__ inline Place(const TileArgs &E, int lane, int b0) {
    const uint32_t stride = (uint32_t)E.B * (uint32_t)sizeof(T);
    // bands past the last are copies of it (their sums are not stored)
    if (E.wide) {
      constexpr int kBands = 16 / (int)sizeof(T);
      pair = lane / kWidePer;
      off = pair * stride +
            (uint32_t)min(b0 + lane % kWidePer * kBands, E.B - kBands) * (uint32_t)sizeof(T);
    } else {
      constexpr int kWords = (int)sizeof(T) / 4;
      pair = kThinPer < 64 ? lane / kThinPer : 0;
      off = pair * stride +
            (uint32_t)min(b0 * kWords + lane % kThinPer, E.B * kWords - 1) * 4u;
    }
  }
};

// Copies what entry en needs into an LDS slot, by direct loads: every wave
// its share of the 64-lane chunks.  Table rows that the atom does not have are
// whatever lies there (the tables are padded by a block): their points and
// rows are masked.
template <typename T, int NB, int NUMAX>
__device__ inline void stage(const TileArgs &E, const TileHead &en, const T *u2, uint32_t slot,
                             int w, int lane, const Place<T, NB> &at) {
  const char *tab = reinterpret_cast<const char *>(E.tab);
  const uint32_t yt = slot + kXRows * table_nfp_c(NUMAX) * 8;
  const uint32_t ut = yt + kYRows * table_nfp_c(NUMAX) * 8;
  const char *xs = tab + (int64_t)en.tab_x * 8;
  const char *ys = tab + (int64_t)en.tab_y * 8;
  const uint32_t off16 = (uint32_t)lane * 16;
  // x rows and y rows: one or two chunks of 1024 bytes each
  if (en.nfp == 8) {
    if (w == 0)
      to_lds<16>(xs, off16, slot);
    else if (w == 1)
      to_lds<16>(ys, off16, yt);
  } else {
    if (w < 2)
      to_lds<16>(xs + w * 1024, off16, slot + w * 1024);
    else
      to_lds<16>(ys + (w - 2) * 1024, off16, yt + (w - 2) * 1024);
  }
  const int np = (en.nu + 1) * (en.nu + 2) / 2;
  const char *src = reinterpret_cast<const char *>(u2 + en.u2 * E.u2_scale);
  const int64_t stride = (int64_t)E.B * sizeof(T);
  if (E.wide) {
    constexpr int kPairs = 64 / Place<T, NB>::kWidePer;  // pairs per chunk
    // (waves from the last on, which had the fewest table rows)
    for (int c = 3 - w; c * kPairs < np; c += 4) {
      const char *s = src + c * kPairs * stride;
      if (c * kPairs + kPairs <= np) {
        to_lds<16>(s, at.off, ut + c * 1024);
      } else if ((int)at.pair < np - c * kPairs) {
        to_lds<16>(s, at.off, ut + c * 1024);
      }
    }
  } else if constexpr (Place<T, NB>::kThinPer <= 64) {
    constexpr int kPairs = 64 / Place<T, NB>::kThinPer;
    for (int c = 3 - w; c * kPairs < np; c += 4)
      if ((int)at.pair < np - c * kPairs)
        to_lds<4>(src + c * kPairs * stride, at.off, ut + c * 256);
  }
}

// a += (phi of lane K of the own 16 lanes) * u: the vector FMA reads the table
// value across lanes, at the rate of a plain one.  (Written out because the
// compiler keeps the broadcast as an instruction of its own.)  A DPP read takes
// two wait states behind a vector instruction that writes the register, which the
// compiler does not see the need of here: a point's first one brings them (and
// volatile keeps it first).  u must not come straight from a matrix instruction:
// settle it.
#define SHO_FMA "v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf"
template <int K, bool kFirst>
__device__ inline void fma_from(double &a, double phi, double u) {
  if constexpr (kFirst)
    asm volatile("s_nop 1\n\t" SHO_FMA : "+v"(a) : "v"(phi), "v"(u), "n"(K));
  else
    asm volatile(SHO_FMA : "+v"(a) : "v"(phi), "v"(u), "n"(K));
}
#undef SHO_FMA
template <int K, int NF, int NB, int N = 0>
__device__ inline void add_point(double (&a)[NB], double phi, const double (&U)[NF][NB]) {
  fma_from<K + N, N == 0>(a[0], phi, U[N][0]);
  if constexpr (NB == 2) fma_from<K + N, false>(a[1], phi, U[N][1]);
  if constexpr (N + 1 < NF) add_point<K, NF, NB, N + 1>(a, phi, U);
}

// The U, written by matrix instructions, may be read by others from here on (the
// last takes up to 18 wait states, which the compiler does not see the need of
// before an asm).  They pass through on both sides of the wait, so that nothing
// that writes them moves down over it and nothing that reads them up.
template <int NF, int NB>
__device__ inline void settle(double (&U)[NF][NB]) {
#pragma unroll
  for (int n = 0; n < NF; ++n)
#pragma unroll
    for (int h = 0; h < NB; ++h) asm volatile("" : "+v"(U[n][h]));
  asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
#pragma unroll
  for (int n = 0; n < NF; ++n)
#pragma unroll
    for (int h = 0; h < NB; ++h) asm volatile("" : "+v"(U[n][h]));
}

// Adds one entry to the wave's 4 rows (4 w + quarter) x 16 points.  range: the
// run of the lane's row within the tile, begin | end << 6; steps: bit t where
// points 2 t, 2 t + 1 are in a run of any of the four.
template <typename T, int NU, int NUMAX, int NB>
__device__ inline void add_entry(const TileArgs &E, uint32_t range, uint32_t steps, int nfp,
                                 const char *slot, int ei, int w, int lane,
                                 double (&acc)[kTileX][NB]) {
  constexpr int NF = NU + 1;
  constexpr int S = (NF + 3) / 4;
  if (steps == 0) return;
  const int q = lane >> 4, i4 = lane & 3;
  const double *yt = reinterpret_cast<const double *>(slot) + kXRows * table_nfp_c(NUMAX) +
                     (4 * w + i4) * nfp + q;
  const Bands<T, NB> *ut = reinterpret_cast<const Bands<T, NB> *>(
      slot + (kXRows + kYRows) * table_nfp_c(NUMAX) * 8);
  // four ny of one nx: quarter q reads pair q; where fewer are left, it reads
  // the last one there is and takes zero instead (the value itself: a zero
  // factor would make NaN of an infinite partial; the table's value is finite
  // in the rows that exist)
  const Bands<T, NB> *um[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) um[m] = ut + min(q, m) * 16 + (lane & 15);
  // y pass: U[nx], quarter = row
  double ay[S];
#pragma unroll
  for (int g = 0; g < S; ++g) ay[g] = yt[4 * g];
  double U[NF][NB];
  int p = 0;
#pragma unroll
  for (int nx = 0; nx < NF; ++nx) {
#pragma unroll
    for (int h = 0; h < NB; ++h) U[nx][h] = 0.0;
#pragma unroll
    for (int g = 0; 4 * g <= NU - nx; ++g) {
      const int left = NU - nx - 4 * g;  // functions after the group's first
      const int m = left < 3 ? left : 3;
      const Bands<T, NB> u = um[m][(p + 4 * g) * 16];
      const bool there = m == 3 || q <= m;
#pragma unroll
      for (int h = 0; h < NB; ++h)
        U[nx][h] = mfma4(ay[g], (double)(there ? u.v[h] : T(0)), U[nx][h]);
    }
    p += NF - nx;
  }
  if (E.phase) {
    // the entry's image T receives e^{-i k.T} times the partials
    const cptr<double> cs = as_const(E.phase) + 2 * ei;
    const double cc = cs[0], sn = cs[1];
#pragma unroll
    for (int n = 0; n < NF; ++n) {
      if constexpr (NB == 2) {
        const double re = U[n][0], im = U[n][1];
        U[n][0] = fma(sn, im, cc * re);
        U[n][1] = fma(-sn, re, cc * im);
      } else {
        U[n][0] = fma((lane & 1) ? -sn : sn, __shfl_xor(U[n][0], 1), cc * U[n][0]);
      }
    }
  }
  // x pass by vector FMAs: all 64 lanes hold a sum of their own, no function is
  // padding, and a point outside the lane's run is switched off.  A register
  // holds phi of kPer points, read one step ahead.
  constexpr int kStep = NF <= 4 ? 4 : 2, kPer = NF <= 4 ? 4 : NF <= 8 ? 2 : 1;
  constexpr int kFn = 16 / kPer, kRegs = kStep / kPer;
  const int j = lane & 15;
  const double *xt = reinterpret_cast<const double *>(slot) + j / kFn * nfp + j % kFn;
  const int lo = (int)(range & 0x3f);
  const uint32_t len = (range >> 6) - (range & 0x3f);
  double ph[2][kRegs];
#pragma unroll
  for (int k = 0; k < kRegs; ++k) ph[0][k] = xt[k * kPer * nfp];
  settle(U);
#pragma unroll
  for (int t = 0; t < kTileX / kStep; ++t) {
    if (t + 1 < kTileX / kStep) {
#pragma unroll
      for (int k = 0; k < kRegs; ++k)
        ph[(t + 1) & 1][k] = xt[((t + 1) * kStep + k * kPer) * nfp];
    }
    if (!(steps >> (t * kStep / 2) & (kStep == 4 ? 3 : 1))) continue;
    auto point = [&](auto at) {
      constexpr int I = decltype(at)::value;
      if ((uint32_t)(t * kStep + I - lo) < len)
        add_point<I % kPer * kFn, NF, NB>(acc[t * kStep + I], ph[t & 1][I / kPer], U);
    };
    point(std::integral_constant<int, 0>{});
    point(std::integral_constant<int, 1>{});
    if constexpr (kStep == 4) {
      point(std::integral_constant<int, 2>{});
      point(std::integral_constant<int, 3>{});
    }
  }
}

// Entries between two barriers, twice as many LDS slots: as many as leave four
// workgroups on a CU (160 KB).  The waves' shares of an entry differ; more of
// them between barriers even out.
constexpr int turn_entries(int numax) { return numax <= 5 ? 2 : 1; }

// Entry records in LDS: chunks of kChunk, and those after them that are staged
// before the chunk ends.  (Scalar loads of the records were waited for where
// they were issued.)
constexpr int kChunk = 8;
constexpr int kRecWords = (int)sizeof(TileEntry) / 4;
constexpr int rec_words(int numax) { return (kChunk + 2 * turn_entries(numax)) * kRecWords; }
static_assert(rec_words(0) <= 2 * kThreads, "two words of the next chunk per thread");

__device__ inline uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

template <typename T, int NUMAX, int NB>
__global__ __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(4))) void k_expand_tiles(TileArgs E,
                                                            const T *__restrict__ u2, T *psi) {
  extern __shared__ char lds[];
  constexpr int kSlot = slot_bytes<T, NB>(NUMAX);
  // Workgroup g runs on XCD g % 8: the band groups of a block one after the
  // other, so that the pieces of a point's row of bands are moved together.
  const uint32_t turn_of = blockIdx.x / kXcds, groups = (uint32_t)E.groups;
  const uint32_t block = turn_of / groups * kXcds + blockIdx.x % kXcds;
  const BlockRec bk = load_uniform(E.blocks + block);
  if (bk.nentries < 0) return;  // padding of the XCD-dealt launch
  const int lane = threadIdx.x & 63, w = wave_id();  // rows 4 w .. 4 w + 3
  const int q = lane >> 4;
  const int b0 = (int)(turn_of % groups) * 16 * NB;
  const int band = b0 + (lane & 15) * NB;
  const Place<T, NB> at(E, lane, b0);
  const int n = bk.nentries;
  // records: a chunk in LDS, this thread's words of the next one in registers
  constexpr int G = turn_entries(NUMAX), kSlots = 2 * G, kRecs = rec_words(NUMAX);
  uint32_t *recs = reinterpret_cast<uint32_t *>(lds + kSlots * kSlot);
  const uint32_t *words = reinterpret_cast<const uint32_t *>(E.entries + bk.entry_begin);
  const int last_word = n * kRecWords - 1, t0 = (int)threadIdx.x, t1 = t0 + kThreads;
  auto chunk_word = [&](int e0, int t) { return words[min(e0 * kRecWords + t, last_word)]; };
  if (t0 < kRecs) recs[t0] = chunk_word(0, t0);
  if (t1 < kRecs) recs[t1] = chunk_word(0, t1);
  uint32_t next0 = chunk_word(kChunk, t0), next1 = t1 < kRecs ? chunk_word(kChunk, t1) : 0u;
  __syncthreads();
  auto head = [&](int i) {  // of record i of the chunk
    const uint32_t *r = recs + i * kRecWords;
    TileHead h;
    h.u2 = (int64_t)((uint64_t)uniform(r[1]) << 32 | uniform(r[0]));
    h.tab_x = (int32_t)uniform(r[2]);
    h.tab_y = (int32_t)uniform(r[3]);
    const uint32_t v = uniform(r[4]);
    h.nu = (int16_t)(v & 0xffff);
    h.nfp = (int16_t)(v >> 16);
    return h;
  };
  const uint32_t lds0 = uniform((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds);
#pragma unroll
  for (int k = 0; k < G; ++k)
    if (k < n) stage<T, NB, NUMAX>(E, head(k), u2, lds0 + k * kSlot, w, lane, at);
  // the wave's values of psi (zeros where there is no point or band)
  const uint32_t bytes_x = (uint32_t)E.B * (uint32_t)sizeof(T);
  const __amdgpu_buffer_rsrc_t rsrc = buffer_of(psi + (int64_t)bk.z * E.ny * E.nx * E.B,
                                                (uint32_t)E.ny * E.nx * bytes_x);
  // Only points of a support are moved (109 x 128 x 122, 197 atoms of cut-off 2,
  // 63 bands: 294 us with whole tiles, 94 so).
  struct Points {
    uint32_t cover, base;
  };
  auto points = [&](int l) {  // of lane l
    const int row = 4 * w + (l >> 4), b = b0 + (l & 15) * NB;
    return Points{b < E.B ? E.cover[block * kTileRows + row] : 0u,
                  (uint32_t)((bk.y0 + row) * E.nx + bk.x0) * bytes_x +
                      (uint32_t)b * (uint32_t)sizeof(T)};
  };
  auto offset = [&](const Points &p, int t) -> uint32_t {
    return p.cover >> t & 1 ? p.base + (uint32_t)t * bytes_x : kOut;
  };
  const Points in = points(lane);
  double acc[kTileX][NB];
  if (E.stream) {
#pragma unroll
    for (int t = 0; t < kTileX; ++t) load_bands<T, NB, 2>(rsrc, offset(in, t), acc[t]);
  } else {
#pragma unroll
    for (int t = 0; t < kTileX; ++t) load_bands<T, NB, 0>(rsrc, offset(in, t), acc[t]);
  }
  // psi is here before the entries begin (known to the compiler, which would
  // else wait for it step by step inside every entry)
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  // Before every G-th entry: the own direct loads of the next G have arrived,
  // after the barrier everybody's have, and nobody reads the slots of the last
  // G any more, which those after the next then fill.
  auto turn = [&](int e) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (e && !(e & (kChunk - 1))) {
      if (t0 < kRecs) recs[t0] = next0;
      if (t1 < kRecs) recs[t1] = next1;
      __syncthreads();
      next0 = chunk_word(e + kChunk, t0);
      if (t1 < kRecs) next1 = chunk_word(e + kChunk, t1);
    }
    const int i = e & (kChunk - 1);
#pragma unroll 1
    for (int k = G; k < 2 * G; ++k)
      if (e + k < n)
        stage<T, NB, NUMAX>(E, head(i + k), u2, lds0 + ((e + k) & (kSlots - 1)) * kSlot, w, lane,
                            at);
  };
  turn(0);
  int e = 0;
  // the current entry: cut-off and table stride, the run of the lane's row, the
  // wave's steps
  const uint32_t *wrec = recs + 6 + 3 * w;
  const uint16_t *rrec = reinterpret_cast<const uint16_t *>(wrec) + q;
  uint32_t kind = uniform(recs[4]), range = rrec[0], steps = uniform(wrec[2]);
  // The entries of a block are sorted by cut-off: one loop per cut-off, so
  // that the accumulators pass through in place (a switch inside one loop had
  // them twice in registers).  The next entry's words are read from LDS before
  // this one is added.
#define X(N)                                                                                  \
  if constexpr (N <= NUMAX) {                                                                 \
    while (e < n && (kind & 0xffff) == N) {                                                   \
      const int o = ((e & (kChunk - 1)) + 1) * kRecWords;                                     \
      const uint32_t k1 = recs[o + 4], r1 = rrec[2 * o], s1 = wrec[o + 2];                    \
      add_entry<T, N, NUMAX, NB>(E, range, steps, kind >> 16,                                 \
                                 lds + (e & (kSlots - 1)) * kSlot, bk.entry_begin + e, w,     \
                                 lane, acc);                                                  \
      kind = uniform(k1);                                                                     \
      range = r1;                                                                             \
      steps = uniform(s1);                                                                    \
      ++e;                                                                                    \
      if (!(e & (G - 1)) && e < n) turn(e);                                                   \
    }                                                                                         \
  }
  SHO_NU_CASES(X)
#undef X
  // (the points are found again, not held in registers across the entries)
  int again = lane;
  asm volatile("" : "+v"(again));
  const Points out = points(again);
  const bool whole = NB == 1 || (E.B & 1) == 0;
#pragma unroll
  for (int t = 0; t < kTileX; ++t) {
    const uint32_t o = offset(out, t);
    if (E.stream) {
      store_bands<T, NB, 2>(rsrc, o, acc[t]);
    } else if (whole) {
      store_bands<T, NB, 0>(rsrc, o, acc[t]);
    } else {
      store_bands<T, 1, 0>(rsrc, o, &acc[t][0]);
      store_bands<T, 1, 0>(rsrc, band + 1 < E.B && o != kOut ? o + (uint32_t)sizeof(T) : kOut,
                           &acc[t][NB - 1]);
    }
  }
}

template <typename T, int NUMAX, int NB>
static hipError_t launch_tiles_nb(const TileArgs &E, const void *u2, void *psi, hipStream_t s) {
  TileArgs args = E;
  args.groups = (E.B + 16 * NB - 1) / (16 * NB);
  if ((uintptr_t)u2 % 16) args.wide = 0;
  hipLaunchKernelGGL((k_expand_tiles<T, NUMAX, NB>),
                     dim3((unsigned)E.nblocks * (unsigned)args.groups), dim3(kThreads),
                     2 * turn_entries(NUMAX) * (slot_bytes<T, NB>(NUMAX)) +
                         rec_words(NUMAX) * 4,
                     s, args, static_cast<const T *>(u2),
                     static_cast<T *>(psi));
  return hipGetLastError();
}

template <typename T, int NUMAX, int NB>
static hipError_t launch_partials_nb(const TileArgs &E, const void *c, void *u2, hipStream_t s) {
  constexpr int NS = (NUMAX + 1) * (NUMAX + 2) * (NUMAX + 3) / 6;
  // An atom's planes in up to four parts where (atom, band group) pairs do not
  // fill the chip: 8 atoms of cut-offs 0..9, 21 bands 16.2 us in one part, 7.7 in
  // four; 6 atoms of cut-off 5, 32 bands 5.4 and 4.5.
  const unsigned groups = (unsigned)((E.B + 16 * NB - 1) / (16 * NB));
  const int64_t wgs = (int64_t)E.natoms_u2 * groups;
  const dim3 g((unsigned)E.natoms_u2, groups, wgs >= 256 ? 1 : wgs >= 128 ? 2 : 4);
  hipLaunchKernelGGL((k_partials<T, NUMAX, NB>), g, dim3(kThreads), NS * 16 * NB * sizeof(T), s,
                     E, static_cast<const T *>(c), static_cast<T *>(u2));
  return hipGetLastError();
}

#define SHO_BUCKETS(F)              \
  if (nu_max <= 3) return F(3);     \
  if (nu_max <= 5) return F(5);     \
  if (nu_max <= 7) return F(7);     \
  if (nu_max <= 9) return F(9);     \
  return F(10);

template <typename T>
static hipError_t tiles_t(int nu_max, const TileArgs &E, const void *u2, void *psi,
                          hipStream_t s) {
  if (E.nb == 1) {
#define F(N) launch_tiles_nb<T, N, 1>(E, u2, psi, s)
    SHO_BUCKETS(F)
#undef F
  }
#define F(N) launch_tiles_nb<T, N, 2>(E, u2, psi, s)
  SHO_BUCKETS(F)
#undef F
}

template <typename T>
static hipError_t partials_t(int nu_max, const TileArgs &E, const void *c, void *u2,
                             hipStream_t s) {
  // two bands per thread where every pair of bands is whole and aligned
  // (cut-off 10: one, the coefficients of two would not fit 64 KB of LDS)
  if (E.B % 2 || ((uintptr_t)c | (uintptr_t)u2) % (2 * sizeof(T)) || E.B < 32 || nu_max > 9) {
#define F(N) launch_partials_nb<T, N, 1>(E, c, u2, s)
    SHO_BUCKETS(F)
#undef F
  }
#define F(N) launch_partials_nb<T, N, 2>(E, c, u2, s)
  SHO_BUCKETS(F)
#undef F
}

}  // namespace tiles

hipError_t launch_tile_partials(int nu_max, bool f32, const TileArgs &E, const void *c, void *u2,
                                hipStream_t s) {
  if (E.natoms_u2 <= 0) return hipSuccess;
  return f32 ? tiles::partials_t<float>(nu_max, E, c, u2, s)
             : tiles::partials_t<double>(nu_max, E, c, u2, s);
}

hipError_t launch_tiles(int nu_max, bool f32, const TileArgs &E, const void *u2, void *psi,
                        hipStream_t s) {
  if (E.nblocks <= 0) return hipSuccess;
  return f32 ? tiles::tiles_t<float>(nu_max, E, u2, psi, s)
             : tiles::tiles_t<double>(nu_max, E, u2, psi, s);
}

}  // namespace sho
