// The propagation of one kz plane of one field in one work-group: forward y
// transforms, forward x, product with the spectrum, inverse x, inverse y, with the
// plane kept in LDS in between. The three separate passes move the plane's padded
// rows through memory four times and its unpadded ones twice; this reads and writes
// the unpadded plane once (10 -> 2 N^2 elements, N = P / 2).
//
// Data are kz-outer, [F][Pz][Nx][Ny], and so is the spectrum, [Hz][Hx][Hy]. Lines
// are transformed by groups of lanes of one wave, several lines per wave, so that a
// line's exchanges need no barrier: LDS operations of a wave are executed in order.
// There are two barriers, between the rows and the columns. A column is exchanged
// within its own N rows of the plane, in two halves (the first half of every
// butterfly's outputs, then the rest), so LDS holds the plane and nothing else.
//
// Needs P_x = P_y = P of two stages, and the plane in 160 KB: P <= 162 for c64 (at 192
// it fits, but the 128 registers that its 12 waves can have spill: 137 us against 115
// of the three passes on a 4.6-lambda sphere), P <= 126 for c128.
//
// Bound by the vector ALU and LDS together (4-lambda sphere with 16 right-hand sides
// in c64: 82% and 50% of the time, measured), with 12 to 20 waves per CU to overlap
// them. The three passes against this one: that sphere 1256 -> 831 us (c64, P = 162);
// 2-lambda sphere with 16 right-hand sides 171 -> 93 us (c64, P = 81); 2.7-lambda
// sphere of third order with three 183 -> 166 us (c128, P = 126).
#pragma once

#include "fft_kernels.h"

namespace aim {
namespace fftk {

template <typename T, class PC, bool FEW = false>
struct PlaneCfg {
  static constexpr int P = PC::P, R0 = PC::r(0), RM = PC::r(PC::ns - 1);
  // R0 = 2 RM: each lane takes two middle butterflies (as the wide x pass)
  static constexpr bool twice = R0 == 2 * RM;
  static constexpr int MB = twice ? 2 : 1;
  static constexpr int TPL = twice ? RM : R0;  // lanes per line
  static constexpr int CB = 64 / TPL;          // lines per wave
  static constexpr int S0 = (R0 + 1) / 2, S1 = (RM + 1) / 2;  // first-half outputs
  static constexpr int N = (P + 1) / 2;        // sources per line at most
  static constexpr int max3(int a, int b, int c) { return a > b ? (a > c ? a : c) : (b > c ? b : c); }
  static constexpr int ROWS = max3(N, S0 * RM, S1 * R0);
  // row length: lane (b, beta) of a column exchange touches element beta LS + b (of a
  // row: b LS + beta), and with LS = CB modulo the 16 (8) elements that an LDS cycle
  // takes, consecutive lanes of a column meet different banks
  static constexpr int kBanks = 128 / (int)sizeof(cx<T>);
  static constexpr int LS = P + ((CB - P) % kBanks + kBanks) % kBanks;
  static constexpr bool same_rows = R0 == RM;
  static constexpr int mid_rows = R0 * (RM - 1), last_rows = same_rows ? 0 : RM * (R0 - 1);
  static constexpr int elems = ROWS * LS + mid_rows + last_rows;
  static constexpr long bytes = (long)elems * (long)sizeof(cx<T>);
  static constexpr bool ok = PC::ns == 2 && P <= 162 && bytes <= 160 * 1024;
  static constexpr int groups_cu = (int)(160 * 1024 / (bytes > 0 ? bytes : 1));
  // waves. Many planes: of 4, 8, 12 and 16, so that a work-group loads the 4 SIMDs of a
  // CU alike (2-lambda sphere with 16 right-hand sides, c64, product: 90 points 5 waves
  // 268 us, 8 waves 222; 81 points 6 waves 205 us, 4 waves 185), the count that keeps
  // most waves busy, i.e. the waves resident (LDS, and registers for 16 to 20 in c64, 8
  // to 10 in c128) times the share of the rounds over row and column tiles in which a
  // wave has a tile. FEW planes: each has a CU to itself and the time is one plane's
  // chain, so the fewest rounds that the registers allow.
  static constexpr int col_tiles = (P + CB - 1) / CB, row_tiles = (N + CB - 1) / CB;
  static constexpr int waves() {
    const int widest = sizeof(T) == 4 ? 16 : 8;
    const int most = sizeof(T) == 4 ? (P < 96 ? 20 : 16) : (P < 81 ? 10 : 8);
    if (!FEW && col_tiles < 4) return col_tiles;
    int best = 1, score = 0;
    for (int w = FEW ? 1 : 4; w <= widest && (w <= col_tiles || !FEW); w += FEW ? 1 : 4) {
      const int rounds = 2 * ((row_tiles + w - 1) / w) + (col_tiles + w - 1) / w;
      const int fit = most / w > 0 ? most / w : 1, groups = groups_cu < fit ? groups_cu : fit;
      // resident waves times busy share, in thousandths
      const int sc = FEW ? 1000 - rounds
                         : groups * 1000 * (2 * row_tiles + col_tiles) / rounds;
      if (sc > score) {
        best = w;
        score = sc;
      }
    }
    return best;
  }
  static constexpr int NW = waves();
};

// Numbers of planes (fields times kz) for which the kernel is the faster one. Up to 90
// points always. Above, few planes leave most CUs without one, and the time is one
// plane's chain, which the separate passes spread over the chip (a flat scatterer
// between grid planes, with one right-hand side 4 P_z planes). The bounds differ with the
// chain: with P = R0 RM a line takes R0 lanes, of which the outer stages use RM (112 = 14
// x 8 and 126 = 14 x 9 divide worst), and in FP64 there is one work-group per CU.
// Product, us, separate -> plane by plane, on scatterers that fill their planes.
// Spheres (P_z = P) with 1, 3, 8 and 16 right-hand sides. c64: P = 81 46 -> 36, 73 -> 57,
// 132 -> 108, 273 -> 188; 96 51 -> 49, 88 -> 84, 188 -> 165, 369 -> 310; 108 60 -> 53, 112 ->
// 105, 272 -> 224, 521 -> 428; 112 64 -> 58, 123 -> 122, 300 -> 272, 531 -> 511; 126 77 ->
// 66, 170 -> 140, 422 -> 339, 776 -> 643; 144 92 -> 92, 228 -> 205, 537 -> 503, 1031 -> 952
// (64 of its 72 nodes: 84 -> 85, 196 -> 176, 466 -> 462, 899 -> 881); 162 142 -> 113, 359 ->
// 281, 861 -> 687, 1684 -> 1298. c128: 48 34 -> 25, 47 -> 43, 74 -> 72, 109 -> 109; 81 62 ->
// 51, 114 -> 89, 257 -> 179, 472 -> 333; 96 72 -> 66, 155 -> 132, 372 -> 299, 646 -> 550; 108
// 94 -> 84, 222 -> 195, 498 -> 443, 925 -> 841; 112 98 -> 94, 235 -> 230, 532 -> 541, 1009 ->
// 1011; 120 115 -> 94, 287 -> 232, 634 -> 552, 1207 -> 1018; 126 133 -> 112, 326 -> 286, 752
// -> 695, 1446 -> 1316. Other lengths up to 120 are faster by 3 to 28%.
// Plates of third order (P_z = 8) with 1, 3 and 8 right-hand sides (32, 96, 256 planes).
// c64: 90 28 -> 23, 37 -> 30, 55 -> 51; 96 28 -> 27, 37 -> 32, 57 -> 57; 112 33 -> 33, 42 ->
// 39, 65 -> 69; 126 35 -> 35, 46 -> 43, 73 -> 73; 144 38 -> 39, 52 -> 48, 85 -> 83; 162 42 ->
// 44, 64 -> 58, 105 -> 98. c128: 90 36 -> 32, 50 -> 44, 76 -> 72; 96 37 -> 38, 51 -> 50, 77 ->
// 80; 108 41 -> 43, 60 -> 57, 92 -> 92; 112 40 -> 50, 59 -> 65, 93 -> 106; 120 42 -> 46, 69 ->
// 66, 103 -> 104; 126 44 -> 53, 75 -> 75, 111 -> 119.
template <typename T, class PC>
constexpr PlaneRange plane_range() {
  constexpr int P = PC::P;
  constexpr bool f32 = sizeof(T) == 4;
  if (!PlaneCfg<T, PC>::ok) return PlaneRange{};
  if (P <= 90) return PlaneRange{1, INT64_MAX};
  if (f32) return PlaneRange{P < 144 ? 32 : 64, INT64_MAX};
  if (P == 112) return PlaneRange{400, 511};  // (a sphere with one right-hand side)
  return PlaneRange{P == 126 ? 300 : 64, INT64_MAX};
}

// Orders LDS accesses of a wave's lanes in the program (the hardware executes a
// wave's LDS operations in order).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename T, class PC, bool FEW>
__global__ void __launch_bounds__((PlaneCfg<T, PC, FEW>::NW * 64))
    k_fft_plane(const cx<T> *__restrict__ in, cx<T> *__restrict__ out, PlaneOut om, int n_x,
                int n_y, int nfield, int Pz, int slots, int Hy, const cx<T> *__restrict__ ghat,
                const cx<T> *__restrict__ tw, const int32_t *__restrict__ yrange,
                FastDiv dfield) {
  using V = cx<T>;
  using C = PlaneCfg<T, PC, FEW>;
  constexpr int P = C::P, R0 = C::R0, RM = C::RM, TPL = C::TPL, CB = C::CB, MB = C::MB,
                LS = C::LS, S0 = C::S0, S1 = C::S1, NW = C::NW;
  // at most P/2 sources and kept outputs per line (even P): upper-half-zero first
  // stages, half of the last outputs
  constexpr bool HALF = R0 % 2 == 0;
  constexpr int NIN = HALF ? R0 / 2 : (R0 + 1) / 2;   // inputs below ceil(P / 2)
  constexpr int NOUT = HALF ? R0 / 2 : (R0 + 1) / 2;
  constexpr uint32_t SV = sizeof(V);
  __shared__ __attribute__((aligned(16))) unsigned char smem[C::bytes];
  V *D = reinterpret_cast<V *>(smem);
  V *twm = D + C::ROWS * LS;                               // middle stage rows
  V *twr = C::same_rows ? twm : twm + C::mid_rows;         // last inverse stage rows

  // work number t = nfield (2 kf + m) + field: folded kz index kf or its mirror,
  // which share a spectrum plane, and their fields get consecutive numbers, and
  // consecutive numbers one XCD
  const int t = (int)(blockIdx.x % kXcd) * slots + (int)(blockIdx.x / kXcd);
  const int tt = (int)fast_div((uint32_t)t, dfield), field = t - tt * nfield;
  const int kf = tt >> 1, m = tt & 1;
  if (2 * kf > Pz) return;  // padding: whole work-groups exit before any barrier
  if (m && (kf == 0 || 2 * kf == Pz)) return;
  const int kz = m ? Pz - kf : kf;
  in += ((int64_t)field * Pz + kz) * n_x * n_y;
  out += field * om.fs + kz * om.zs;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const V zero = mk<V>((T)0, (T)0);
  // the first forward stage of a line: butterfly beta < RM, inputs beta + q RM
  auto first_stage = [&](V *v) AIM_AI {
    if constexpr (HALF) {
      dft_upper_zero<R0, false, V>(v);
    } else {
      static_for<R0 - NIN>([&](auto q_) AIM_AI { v[NIN + decltype(q_)::value] = zero; });
      Dft<R0, false, V>::run(v);
    }
  };
  // twiddles and the last forward stage of middle butterfly j
  auto middle_stage = [&](V *v, int j) AIM_AI {
    const V *row = twm + j * (RM - 1);
    static_for<RM - 1>([&](auto q_) AIM_AI {
      constexpr int q = decltype(q_)::value + 1;
      v[q] = tw_mul<false>(v[q], row, q - 1);
    });
    Dft<RM, false, V>::run(v);
  };

  // consecutive lanes hold consecutive rows (then their LDS rows, LS apart, meet
  // consecutive groups of banks)
  const int rb = lane / CB, rr = lane - rb * CB;
  // (buffer accesses at kOutside, beyond the resource, read zero and store nothing:
  // no branch per element)
  constexpr uint32_t kOutside = 0x80000000u;
  const __amdgpu_buffer_rsrc_t rin = buffer_of(in, (uint32_t)(n_x * n_y) * SV);
  auto row_range = [&](int row, int &lo, int &hi) AIM_AI {
    lo = yrange ? yrange[2 * row] : 0;
    hi = yrange ? min(n_y, yrange[2 * row + 1]) : n_y;
  };
  auto load_row = [&](V *v, int row) AIM_AI {
    if (rb >= RM || row >= n_x) return;
    int lo, hi;
    row_range(row, lo, hi);
    static_for<NIN>([&](auto q_) AIM_AI {
      constexpr int q = decltype(q_)::value;
      const int i = rb + q * RM;
      v[q] = bload<V>(rin, (i >= lo && i < hi) ? (uint32_t)(row * n_y + i) * SV : kOutside, 0u);
    });
  };
  V v[R0];
  load_row(v, wave * CB + rr);  // in flight while the tables are filled

  for (int i = threadIdx.x; i < C::mid_rows; i += 64 * NW) {
    const int jj = i / (RM - 1), q = i - jj * (RM - 1) + 1;
    twm[i] = tw[jj * q];
  }
  if constexpr (!C::same_rows)
    for (int i = threadIdx.x; i < C::last_rows; i += 64 * NW) {
      const int jj = i / (R0 - 1), q = i - jj * (R0 - 1) + 1;
      twr[i] = tw[jj * q];
    }
  __syncthreads();

  // forward y transforms of the rows
  for (int r0 = wave * CB; r0 < n_x; r0 += NW * CB) {
    const int row = r0 + rr;
    const bool ok = rb < TPL && row < n_x;
    V *Dr = D + row * LS;
    if (r0 != wave * CB) load_row(v, row);
    if (ok && rb < RM) {
      first_stage(v);
      static_for<R0>([&](auto p_) AIM_AI {
        constexpr int p = decltype(p_)::value;
        Dr[p * RM + rb] = v[p];
      });
    }
    wave_sync();
    V u[MB][RM];
    static_for<MB>([&](auto k_) AIM_AI {
      constexpr int k = decltype(k_)::value;
      const int j = rb + TPL * k;
      if (ok)
        static_for<RM>([&](auto q_) AIM_AI {
          constexpr int q = decltype(q_)::value;
          u[k][q] = Dr[j * RM + q];
        });
    });
    wave_sync();
    static_for<MB>([&](auto k_) AIM_AI {
      constexpr int k = decltype(k_)::value;
      const int j = rb + TPL * k;
      if (ok) {
        middle_stage(u[k], j);
        static_for<RM>([&](auto p_) AIM_AI {
          constexpr int p = decltype(p_)::value;
          Dr[p * R0 + j] = u[k][p];
        });
      }
    });
  }
  __syncthreads();

  // the columns: forward x, spectrum, inverse x
  const int beta = lane / CB, b = lane - beta * CB;
  const int gplane = Hy * (P / 2 + 1);
  const __amdgpu_buffer_rsrc_t gres =
      buffer_of(ghat + (int64_t)kf * gplane, (uint32_t)gplane * SV);
  for (int c0 = wave * CB; c0 < P; c0 += NW * CB) {
    const int c = c0 + b;
    const bool ok = beta < TPL && c < P;
    const bool okb = ok && beta < RM;
    V *Dc = D + c;
    if (okb)
      static_for<NIN>([&](auto q_) AIM_AI {
        constexpr int q = decltype(q_)::value;
        const int i = beta + q * RM;
        v[q] = i < n_x ? Dc[i * LS] : zero;
      });
    wave_sync();
    if (okb) first_stage(v);
    const int fky = (c <= P - c) ? c : P - c;
    V u[MB][RM];
    static_for<2>([&](auto h_) AIM_AI {
      constexpr int h = decltype(h_)::value, p0 = h ? S0 : 0, p1 = h ? R0 : S0;
      if (okb)
        static_for<p1 - p0>([&](auto p_) AIM_AI {
          constexpr int p = decltype(p_)::value;
          Dc[(p * RM + beta) * LS] = v[p0 + p];
        });
      wave_sync();
      static_for<MB>([&](auto k_) AIM_AI {
        constexpr int k = decltype(k_)::value;
        if constexpr (!C::twice || k == h) {
          const int j = beta + TPL * k;
          if (ok && (C::twice || (h ? j >= S0 : j < S0)))
            static_for<RM>([&](auto q_) AIM_AI {
              constexpr int q = decltype(q_)::value;
              u[k][q] = Dc[((h ? j - S0 : j) * RM + q) * LS];
            });
        }
      });
      wave_sync();
    });
    static_for<MB>([&](auto k_) AIM_AI {
      constexpr int k = decltype(k_)::value;
      const int j = beta + TPL * k;
      if (ok) {
        // kx = j + R0 p, folded at P / 2 (at run time for the middle p of an odd RM)
        V g[RM];
        const uint32_t g_lo = (uint32_t)(j * Hy + fky) * SV;
        const uint32_t g_hi = (uint32_t)((R0 - 1 - j) * Hy + fky) * SV;
        static_for<RM>([&](auto p_) AIM_AI {
          constexpr int p = decltype(p_)::value;
          if constexpr (2 * p <= RM - 2) {
            g[p] = bload<V>(gres, g_lo, (uint32_t)(R0 * p * Hy) * SV);
          } else if constexpr (2 * p >= RM) {
            g[p] = bload<V>(gres, g_hi, (uint32_t)((P - R0 * p - R0 + 1) * Hy) * SV);
          } else {
            const int kx = j + R0 * p;
            g[p] = bload<V>(gres, (uint32_t)((kx <= P - kx ? kx : P - kx) * Hy + fky) * SV, 0u);
          }
        });
        middle_stage(u[k], j);
        static_for<RM>([&](auto p_) AIM_AI {
          constexpr int p = decltype(p_)::value;
          u[k][p] = cmul(u[k][p], g[p]);
        });
        Dft<RM, true, V>::run(u[k]);
      }
    });
    V w[R0];
    static_for<2>([&](auto h_) AIM_AI {
      constexpr int h = decltype(h_)::value, p0 = h ? S1 : 0, p1 = h ? RM : S1;
      static_for<MB>([&](auto k_) AIM_AI {
        constexpr int k = decltype(k_)::value;
        const int j = beta + TPL * k;
        if (ok)
          static_for<p1 - p0>([&](auto p_) AIM_AI {
            constexpr int p = decltype(p_)::value;
            Dc[(p * R0 + j) * LS] = u[k][p0 + p];
          });
      });
      wave_sync();
      if (okb && (h ? beta >= S1 : beta < S1))
        static_for<R0>([&](auto q_) AIM_AI {
          constexpr int q = decltype(q_)::value;
          w[q] = Dc[((h ? beta - S1 : beta) * R0 + q) * LS];
        });
      wave_sync();
    });
    auto st = [&](int i, V x) AIM_AI {
      if (i < n_x) Dc[i * LS] = x;
    };
    if (okb) stage_compute_store_p<R0, true, false, NOUT, true>(w, beta, RM, 1, twr, st);
  }
  __syncthreads();

  // inverse y transforms of the rows
  const __amdgpu_buffer_rsrc_t rout =
      buffer_of(out, (uint32_t)((n_x - 1) * om.xs + (n_y - 1) * om.ys + 1) * SV);
  for (int r0 = wave * CB; r0 < n_x; r0 += NW * CB) {
    const int row = r0 + rr;
    const bool ok = rb < TPL && row < n_x;
    V *Dr = D + row * LS;
    V u[MB][RM];
    static_for<MB>([&](auto k_) AIM_AI {
      constexpr int k = decltype(k_)::value;
      const int j = rb + TPL * k;
      if (ok)
        static_for<RM>([&](auto q_) AIM_AI {
          constexpr int q = decltype(q_)::value;
          u[k][q] = Dr[j + q * R0];
        });
    });
    wave_sync();
    static_for<MB>([&](auto k_) AIM_AI {
      constexpr int k = decltype(k_)::value;
      const int j = rb + TPL * k;
      if (ok) {
        Dft<RM, true, V>::run(u[k]);
        static_for<RM>([&](auto p_) AIM_AI {
          constexpr int p = decltype(p_)::value;
          Dr[p * R0 + j] = u[k][p];
        });
      }
    });
    wave_sync();
    if (ok && rb < RM) {
      int lo, hi;
      row_range(row, lo, hi);
      V w[R0];
      static_for<R0>([&](auto q_) AIM_AI {
        constexpr int q = decltype(q_)::value;
        w[q] = Dr[rb * R0 + q];
      });
      auto st = [&](int i, V x) AIM_AI {
        bstore<V>(x, rout,
                  (i >= lo && i < hi) ? (uint32_t)(row * om.xs + i * om.ys) * SV : kOutside, 0u);
      };
      stage_compute_store_p<R0, true, false, NOUT, true>(w, rb, RM, 1, twr, st);
    }
  }
}

// z passes into and out of kz-outer grids [F][Pz][Nx Ny]: forward from the projected
// sources [F][Nx Ny][Nz], inverse to the field-interleaved grid [Nx Ny][Nz][F] that
// the interpolation reads; few nodes of these two are occupied. A work-group takes B
// occupied lines of one field, lanes along the lines, so the kz-outer side moves in
// runs of 256 bytes (lanes along the transform, as in k_fft_contig, would touch one
// element per cache line). Bound by that side's traffic: 4-lambda sphere with 16
// right-hand sides in c64 (571 MB), forward 140 us, inverse 158 us (3.6 TB/s).
template <typename T, class PC>
constexpr int tile_zplane() {
  int B = 256 / (int)sizeof(cx<T>);
  while (B > 4 && (PC::maxnb() * B > 1024 ||
                   (long)PC::P * (B + 1) * (long)sizeof(cx<T>) > kLdsBudget))
    B /= 2;
  return B;
}
template <typename T, bool INV, bool PR, class PC>
__global__ void __launch_bounds__((round_up_c(PC::maxnb() * tile_zplane<T, PC>(), 64)))
    k_fft_zplane(const cx<T> *__restrict__ in, cx<T> *__restrict__ out, int n_in, int n_out,
                 int64_t nl, const int32_t *__restrict__ sel, const int32_t *__restrict__ range,
                 int64_t A1, int nfield, const cx<T> *__restrict__ tw, int64_t slots,
                 FastDiv dmin) {
  using V = cx<T>;
  constexpr int P = PC::P, B = tile_zplane<T, PC>();
  __shared__ V lds[PC::ns > 1 ? P * (B + 1) : 1];
  V *twl = lds + (PC::ns > 1 ? P * B : 0);
  // work number, consecutive ones on one XCD: forward line tiles of a field; inverse
  // fields of a line tile, whose stores interleave
  const int64_t vb = (int64_t)(blockIdx.x % kXcd) * slots + blockIdx.x / kXcd;
  const uint32_t hi_ = fast_div((uint32_t)vb, dmin), lo_ = (uint32_t)vb - hi_ * dmin.d;
  const int field = (int)(INV ? lo_ : hi_);
  const int64_t tile = INV ? hi_ : lo_;
  if (field >= nfield || tile * B >= nl) return;  // the whole work-group
  const int b = threadIdx.x % B, beta = threadIdx.x / B;
  const int64_t l = tile * B + b;
  const bool line_ok = l < nl;
  const int64_t line = sel[line_ok ? l : nl - 1];
  const int32_t *rg = range + 4 * (line_ok ? l : nl - 1);
  // sources (forward) and the interpolation's nodes (inverse) lie in [lo, g0) and
  // [g1, hi) of the line
  const int lo = rg[0], g0 = rg[1], g1 = rg[2], hi = min(rg[3], INV ? n_out : n_in);
  const V *gin = INV ? in + (int64_t)field * n_in * A1 + line
                     : in + ((int64_t)field * A1 + line) * n_in;
  V *gout = INV ? out + line * (int64_t)n_out * nfield + field
                : out + (int64_t)field * n_out * A1 + line;
  const int es_in = INV ? (int)A1 : 1, es_out = INV ? nfield : (int)A1;
  if constexpr (PC::ns > 1) {
    for (int i = threadIdx.x; i < P; i += blockDim.x) twl[i] = tw[i];
    __syncthreads();
  }
  static_for<PC::ns>([&](auto s_) AIM_AI {
    constexpr int s = decltype(s_)::value;
    constexpr int R = PC::r(s), L = PC::lb(s), Mp = P / (L * R), nb = P / R;
    constexpr bool first = (s == 0), last = (s == PC::ns - 1);
    const bool active = line_ok && (beta < nb);
    auto inside = [&](int i) AIM_AI { return i >= lo && i < hi && (i < g0 || i >= g1); };
    auto ld = [&](int i) AIM_AI -> V {
      if constexpr (first)
        return (INV ? i < n_in : inside(i)) ? gin[i * es_in] : mk<V>((T)0, (T)0);
      else return lds[i * B + b];
    };
    auto st = [&](int i, V v) AIM_AI {
      if constexpr (last) {
        if (INV ? inside(i) : i < n_out) gout[i * es_out] = v;
      } else {
        lds[i * B + b] = v;
      }
    };
    constexpr bool uz = stage_uz<R, INV, PR, first, last>();
    constexpr int nout = stage_nout<R, INV, PR, first, last>();
    V v[R];
    if (active) {
      if constexpr (uz) stage_load_p<R, R / 2, V>(v, beta, Mp, ld);
      else stage_load<R, INV, V>(v, beta, Mp, ld);
    }
    if constexpr (!first && !last) __syncthreads();
    if (active) stage_compute_store_p<R, INV, uz, nout, false>(v, beta, L, Mp, twl, st);
    if constexpr (!last) __syncthreads();
  });
}

// planes up to which each gets the widest work-group (2-lambda sphere in c64, 324
// planes: 17.8 -> 14.9 us; in c128 23.5 -> 26 us, so only below one plane per CU;
// 3-lambda sphere in c64, 504 planes: 32.6 -> 34.9 us; a 3-lambda plate's 4 planes: 12.1
// -> 8.5 us)
template <typename T>
constexpr int64_t kFewPlanes = sizeof(T) == 4 ? 384 : 256;
template <typename T, class PC>
void launch_plane(const cx<T> *in, cx<T> *out, const PlaneOut &om, int Nx, int Ny, int F, int Pz,
                  int Hy, const cx<T> *ghat, const cx<T> *tw, const int32_t *yrange,
                  hipStream_t s) {
  using C = PlaneCfg<T, PC>;
  if constexpr (plane_range<T, PC>().any()) {
    if (Nx < 1 || Ny < 1 || 2 * Nx > PC::P + 1 || 2 * Ny > PC::P + 1 ||
        (PC::P % 2 == 0 && (2 * Nx > PC::P || 2 * Ny > PC::P)) || Hy != PC::P / 2 + 1)
      throw Error(AIM_ERR_ARG, "plane pass: more than P/2 sources on a line");
    if (om.xs < 0 || om.ys < 0 ||
        ((int64_t)(Nx - 1) * om.xs + (int64_t)(Ny - 1) * om.ys + 1) * (int64_t)sizeof(cx<T>) >
            INT32_MAX)
      throw Error(AIM_ERR_ARG, "plane pass: a plane's output beyond 32-bit offsets");
    const int64_t items = 2 * ((int64_t)Pz / 2 + 1) * F;
    const int64_t slots = (items + kXcd - 1) / kXcd;
    if (slots * kXcd > INT32_MAX) throw Error(AIM_ERR_ARG, "plane pass: too many planes");
    auto go = [&](auto few_) {
      constexpr bool FEW = decltype(few_)::value;
      hipLaunchKernelGGL((k_fft_plane<T, PC, FEW>), dim3((unsigned)(slots * kXcd)),
                         dim3(64 * PlaneCfg<T, PC, FEW>::NW), 0, s, in, out, om, Nx, Ny, F, Pz,
                         (int)slots, Hy, ghat, tw, yrange, make_fastdiv((uint32_t)F));
    };
    if (PlaneCfg<T, PC, true>::NW != C::NW && (int64_t)F * Pz <= kFewPlanes<T>)
      go(std::bool_constant<(PlaneCfg<T, PC, true>::NW != C::NW)>{});
    else
      go(std::false_type{});
    LAUNCHCHECK();
  } else {
    bad_length(PC::P);
  }
}

// lengths with a z pass between kz-outer grids
template <class PC>
constexpr bool zplane_ok() {
  return PC::P <= 576;
}
template <typename T, class PC>
void launch_zplane(const cx<T> *in, cx<T> *out, int n_in, int n_out, int F, int64_t nl,
                   const int32_t *sel, const int32_t *range, int64_t A1, bool inverse,
                   const cx<T> *tw, hipStream_t s) {
  if constexpr (zplane_ok<PC>()) {
    constexpr int B = tile_zplane<T, PC>(), threads = round_up_c(PC::maxnb() * B, 64);
    if ((int64_t)std::max(n_in, n_out) * std::max<int64_t>(A1, F) > INT32_MAX)
      throw Error(AIM_ERR_ARG, "z pass: grid beyond 32-bit offsets");
    const int64_t tiles = (nl + B - 1) / B, blocks = tiles * F, slots = (blocks + kXcd - 1) / kXcd;
    if (slots * kXcd > INT32_MAX) throw Error(AIM_ERR_ARG, "z pass: too many lines");
    const bool pr = pass_prunable<PC>(inverse, n_in, n_out);
    auto go = [&](auto kern) {
      hipLaunchKernelGGL(kern, dim3((unsigned)(slots * kXcd)), dim3(threads), 0, s, in, out, n_in,
                         n_out, nl, sel, range, A1, F, tw, slots,
                         make_fastdiv((uint32_t)(inverse ? F : tiles)));
    };
    if (inverse)
      pr ? go(k_fft_zplane<T, true, true, PC>) : go(k_fft_zplane<T, true, false, PC>);
    else
      pr ? go(k_fft_zplane<T, false, true, PC>) : go(k_fft_zplane<T, false, false, PC>);
    LAUNCHCHECK();
  } else {
    bad_length(PC::P);
  }
}

}  // namespace fftk
}  // namespace aim
