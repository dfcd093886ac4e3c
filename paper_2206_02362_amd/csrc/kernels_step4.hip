// Up to four leapfrog time steps per launch, for grids too small to fill the
// device.  Same recursion and the same operations per cell as the one- and
// two-step kernels, and the same bits (in extended precision through the shared
// df_update and df_low_laplacian).
//
// What bounds these grids is not work but the launch: a 100 x 200 model with
// one shot is 36 two-step workgroups, and a two-step launch took 7.5 us
// whatever was computed in it (dispatch, and a chain of cold loads, as every
// launch starts with an empty L2).  Four steps per launch halve the number of
// launches, and small tiles (40 rows x 8 columns, 8 wavefronts) keep the
// serial work of a workgroup short: the halo of 12 cells is recomputed by the
// neighbours, work that the idle compute units have room for.  Measured,
// 1500 steps: 6.0 ms with two steps per launch, 2.8 ms with four; a launch
// takes 7 to 8 us, its vector units busy 14-18 % and its wavefronts waiting for
// memory half of their cycles.
//
// What a launch waits for is a chain of loads, so nothing with an address
// known from the arguments waits behind something else: the list ranges and
// the tapers are read ahead of the tile, the tile's bounds are masks without
// branches, and the tile's coordinates come from multiplications.  Against
// loads where their values are used: variable-projection step of 100 x 200
// with two shots 41.1 -> 39.8 ms, its gradient with one shot 14.2 -> 13.4 ms.
//
// A workgroup stages u^n on its tile plus a 16-cell halo in LDS and computes
// u^{n+1} on the tile plus 12 cells, u^{n+2} on the tile plus 8, and so on,
// alternating between two LDS tiles (one barrier per step).  Lane = row
// z0 - 12 + lane for every step; wavefront w keeps the same W columns
// throughout, so V, the taper and the field one step back (the previous
// step's centre value) stay in registers.  Cells outside the shrinking valid
// region hold values nobody reads for a result: a valid cell's operands are
// valid, so they are computed or not as is convenient (a wavefront whose
// columns are all outside skips the step).
//
// The update is written with its fused multiply-adds spelled out, in the form
// that the two-step kernel compiles to, and contraction is off: the bits do
// not depend on how the compiler splits the steps into blocks.
//
// Fields of the steps are written where out[s] is given: a field ring's last
// two, or every step of a time ring.
#include "internal.h"

#include <type_traits>

#pragma clang fp contract(off)

namespace fw {

constexpr int kT = kMaxSteps;

template <int TX, bool DF>
struct Step4Tile {
  static constexpr int C0 = TX + 8 * kT;       // u^n columns x0 - 16 .. x0 + TX + 15
  static constexpr int ROWS = 72;              // rows z0 - 16 .. z0 + 55
  float u[2][C0][ROWS];
};
template <int TX>
struct Step4Tile<TX, true> : Step4Tile<TX, false> {
  unsigned short l[2][Step4Tile<TX, false>::C0][Step4Tile<TX, false>::ROWS];
};

template <int TX, int MODE>
__global__ void __launch_bounds__(64 * kWaves4) k_step4(const Step4Args a) {
  constexpr bool T2 = (MODE & kModeT2) != 0;
  constexpr bool DS = (MODE & kModeDsrc) != 0;
  constexpr bool NU = (MODE & kModeNu) != 0;
  constexpr bool DF = (MODE & kModeDF) != 0;
  constexpr bool FS = (MODE & kModeFS) != 0;
  constexpr bool PS = !DS && !NU;              // a dense source and point sources exclude each other
  using Tile = Step4Tile<TX, DF>;
  constexpr int C0 = Tile::C0, ROWS = Tile::ROWS;
  constexpr int C1 = TX + 2 * kHalo4;          // columns computed in the first step
  constexpr int W = C1 / kWaves4;              // columns per wavefront
  constexpr int NC = C0 / kWaves4;             // tile columns loaded per wavefront
  static_assert(C1 % kWaves4 == 0 && C0 % kWaves4 == 0 && C0 % 8 == 0, "tile width");
  __shared__ Tile sh;

  warm_args<sizeof(Step4Args)>();
  const int total = a.ntz * a.ntx * a.nshots;
  const int per = (total + 7) >> 3;
  const int logical = (blockIdx.x & 7) * per + (blockIdx.x >> 3);    // XCD-contiguous tile ranges
  if (logical >= total) return;
  const int strip = (int)a.by_ntz.div((unsigned)logical), tzi = logical - strip * a.ntz;
  const int s = (int)a.by_ntx.div((unsigned)strip), txi = strip - s * a.ntx;
  const int z0 = tzi * kTZ4, x0 = txi * TX;
  const int NZ = a.NZ, NX = a.NX, LZ = a.LZ;
  const int CB = LZ * 4;
  const unsigned FB = (unsigned)NX * (unsigned)CB;
  const long soff = (long)s * a.sstride;
  const auto r_cur = rsrc(a.cur + soff, FB);
  const auto r_prev = rsrc(a.prev + soff, FB);
  const auto r_V = rsrc(a.V, FB);
  [[maybe_unused]] __amdgpu_buffer_rsrc_t r_lcur, r_lprev;
  if constexpr (DF) {
    r_lcur = rsrc(a.lo_cur + soff, FB / 2);
    r_lprev = rsrc(a.lo_prev + soff, FB / 2);
  }

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int z = z0 - kHalo4 + lane;
  const bool zin = z >= 0 && z < NZ;
  const bool zown = lane >= kHalo4 && lane < kHalo4 + kTZ4;
  const int vz_st = zin && zown ? z * 4 : kOutOfRange;       // rows stored
  [[maybe_unused]] const int vz16_st = zin && zown ? z * 2 : kOutOfRange;
  const int vzc = min(max(z, 0), NZ - 1) * 4;                // clamped row
  const int xs = x0 - kHalo4 + w * W;                        // this wavefront's first column

  // list ranges of the point sources and the receivers and the tapers: scalar
  // loads that only need the arguments, ahead of everything that waits
  int i0 = 0, i1 = 0;
  if constexpr (PS) {
    i0 = a.inj.ptr[logical * kWaves4 + w];
    i1 = a.inj.ptr[logical * kWaves4 + w + 1];
  }
  const int *ranges = a.ext.ptr ? a.ext.ptr + logical : reinterpret_cast<const int *>(a.gx);
  const int e0 = ranges[0], en0 = ranges[1];
  float gxc[W];
#pragma unroll
  for (int j = 0; j < W; ++j) gxc[j] = a.gx[min(max(xs + j, 0), NX - 1)];
  const float gzc = a.gz[vzc / 4];                           // taper at the clamped row (nonzero)

  // u^n tile: lane = row z0 - 16 + lane of a column, then the last 8 rows of
  // 8 columns per wavefront; cells outside the grid read zero
  float v[NC], vt;
  [[maybe_unused]] unsigned short l[NC], lt;
  [[maybe_unused]] float sg = 1.f, sgt = 1.f;
  {
    const int zt = z0 - 4 * kT + lane, ztt = z0 - 4 * kT + 64 + (lane & 7);
    int zr = zt, zrt = ztt;
    if constexpr (FS) {
      zr = fs_mirror_row(zt, a.fs, sg);
      zrt = fs_mirror_row(ztt, a.fs, sgt);
    }
    const bool zt_in = zt >= 0 && zt < NZ;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int x = x0 - 4 * kT + w + kWaves4 * i;
      const bool in = (x >= 0) & (x < NX) & zt_in;           // no short cut: no branch
      const int o = in ? x * CB + zr * 4 : kOutOfRange;
      v[i] = ld(r_cur, o, 0);
      if constexpr (DF) l[i] = ld16(r_lcur, o == kOutOfRange ? kOutOfRange : o / 2, 0);
    }
    const int ct = w * 8 + (lane >> 3), xt = x0 - 4 * kT + ct;
    const bool in = (ct < C0) & (xt >= 0) & (xt < NX) & (ztt >= 0) & (ztt < NZ);
    const int o = in ? xt * CB + zrt * 4 : kOutOfRange;
    vt = ld(r_cur, o, 0);
    if constexpr (DF) lt = ld16(r_lcur, o == kOutOfRange ? kOutOfRange : o / 2, 0);
  }
  // own-cell operands, read at the nearest cell inside the grid
  float pv[W], vv[W], g[W];
  [[maybe_unused]] unsigned short pl[W];
#pragma unroll
  for (int j = 0; j < W; ++j) {
    const int xc = min(max(xs + j, 0), NX - 1);
    pv[j] = ld(r_prev, vzc, xc * CB);
    vv[j] = ld(r_V, vzc, xc * CB);
    if constexpr (DF) pl[j] = ld16(r_lprev, vzc / 2, xc * (CB / 2));
  }
  // dense sources of every step (Dsrc), or the e slots k + 1, k, k - 1, ...
  [[maybe_unused]] float dn[NU ? kT + 2 : kT][W];
  if constexpr (DS || NU) {
    const int vze = z >= a.ez0 && z < a.ez1 ? vzc : kOutOfRange;
#pragma unroll
    for (int q = 0; q < (NU ? kT + 2 : kT); ++q) {
      // slots past the last step are not given: any slot stands in for them
      const auto r = rsrc((a.ds[q] ? a.ds[q] : a.ds[0]) + (long)s * a.ds_sstride, FB);
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const int xc = min(max(xs + j, 0), NX - 1);
        dn[q][j] = ld(r, xc >= a.ex0 && xc < a.ex1 ? vze : kOutOfRange, xc * CB);
      }
    }
  }
  // point sources of this wavefront's columns: entries and the samples of
  // every step, behind the tile loads
  const int cnt = i1 - i0;
  [[maybe_unused]] int2 en = {0, 0};
  [[maybe_unused]] float sv[kT] = {};
  auto sample = [&](int st) {
    return a.inj.val[(long)en.y * a.inj.stride_idx + a.inj.t + st * a.inj_dt] * a.inj.scale;
  };
  if constexpr (PS) {
    if (lane < cnt) {
      en = a.inj.ent[i0 + lane];
#pragma unroll
      for (int st = 0; st < kT; ++st)
        if (st < a.steps) sv[st] = sample(st);
    }
  }
  const int e1 = a.ext.ptr ? en0 : e0;
  int2 first = {0, 0};                                       // this thread's first receiver
  if (e0 + tid < e1) first = a.ext.ent[e0 + tid];
#pragma unroll
  for (int j = 0; j < W; ++j) g[j] = (zin ? gzc : 0.f) * gxc[j];

#pragma unroll
  for (int i = 0; i < NC; ++i) {
    sh.u[0][w + kWaves4 * i][lane] = FS ? sg * v[i] : v[i];
    if constexpr (DF) sh.l[0][w + kWaves4 * i][lane] = FS && sg < 0.f ? (unsigned short)(l[i] ^ 0x8000u) : l[i];
  }
  if (w * 8 < C0) {                                          // wave-uniform
    sh.u[0][w * 8 + (lane >> 3)][64 + (lane & 7)] = FS ? sgt * vt : vt;
    if constexpr (DF)
      sh.l[0][w * 8 + (lane >> 3)][64 + (lane & 7)] = FS && sgt < 0.f ? (unsigned short)(lt ^ 0x8000u) : lt;
  }

  const int lz = lane + kR;                                  // LDS row of this lane's row
  const int cl = w * W + kR;                                 // LDS column of this wavefront's first column
  [[maybe_unused]] const bool fs_near = FS && a.fs >= 0 && z0 - kHalo4 <= a.fs - 1 && z0 - kHalo4 + 63 >= a.fs - kR;
  [[maybe_unused]] float c0l = 0.f;
  if constexpr (DF) {
#pragma unroll
    for (int k = 0; k < kR; ++k) c0l -= 2.f * (a.cz[k] + a.cx[k]);
  }

  // one step; ST as a constant, so that everything a step picks by it is fixed
  auto step = [&](auto ST) __attribute__((always_inline)) {
    constexpr int st = decltype(ST)::value;
    float(*cur)[ROWS] = sh.u[st & 1], (*nxt)[ROWS] = sh.u[(st + 1) & 1];
    [[maybe_unused]] unsigned short(*lcur)[ROWS] = nullptr, (*lnxt)[ROWS] = nullptr;
    if constexpr (DF) {
      lcur = sh.l[st & 1];
      lnxt = sh.l[(st + 1) & 1];
    }
    __syncthreads();
    // receivers of u^{n+st}
    for (int e = e0 + tid; e < e1; e += 64 * kWaves4) {
      const int2 rc = e == e0 + tid ? first : a.ext.ent[e];
      a.ext.out[(long)rc.y * a.ext.stride_idx + a.ext.t + st] = cur[(rc.x >> 6) + 4 * kT][(rc.x & 63) + 4 * kT];
    }
    // columns still valid after this step: 4 st .. C1 - 4 st - 1
    if (w * W + W <= 4 * st || w * W >= C1 - 4 * st) return;

    float src[W];
#pragma unroll
    for (int j = 0; j < W; ++j) src[j] = DS ? dn[st][j] : 0.f;
    if constexpr (NU) {
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const float gn = gzc * gxc[j];
        src[j] += fmaf(gn, dn[st][j], fmaf(-2.f, dn[st + 1][j], dn[st + 2][j] / gn));
      }
    }
    if constexpr (PS) {
      if (cnt > 0) {                                         // wave-uniform
        if (__builtin_amdgcn_readfirstlane(en.x) & kInjRepeat) {
          for (int b = 0; b < cnt; b += 64) {
            if (cnt > 64 && b + lane < cnt) en = a.inj.ent[i0 + b + lane];
            const float val = cnt > 64 ? (b + lane < cnt ? sample(st) : 0.f) : sv[st];
            const int n = min(64, cnt - b);
            for (int k = 0; k < n; ++k) {
              const int kx = __builtin_amdgcn_readlane(en.x, k) & ~kInjRepeat;
              const float kv = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, val), k));
              if ((kx & 63) == lane) {
#pragma unroll
                for (int jj = 0; jj < W; ++jj)
                  if (jj == kx >> 6) src[jj] += kv;
              }
            }
          }
        } else {
          // through this wavefront's own columns of the next tile, not yet written
          float(*own)[ROWS] = nxt + cl;
          add_through_lds(own, lane, src, [&]() {
            for (int b = 0; b < cnt; b += 64) {
              if (cnt > 64 && b + lane < cnt) en = a.inj.ent[i0 + b + lane];
              if (b + lane < cnt) own[en.x >> 6][en.x & 63] = cnt > 64 ? sample(st) : sv[st];
            }
          });
        }
      }
    }

    const float *base = &cur[cl][lz];
    [[maybe_unused]] const unsigned short *basel = nullptr;
    if constexpr (DF) basel = &lcur[cl][lz];
    const bool keep = a.out[st] != nullptr;                  // uniform
    float dxf[kR][W];                                        // forward x-differences, as in the two-step kernel
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const float *col = base + j * ROWS;
      const float c = col[0];
      float lap = 0.f;
      [[maybe_unused]] double lapd = 0.0;
#pragma unroll
      for (int k = 1; k <= kR; ++k) {
        dxf[k - 1][j] = col[k * ROWS] - c;
        const float back = j >= k ? -dxf[k - 1][j - k] : col[-k * ROWS] - c;
        if constexpr (DF) {
          lapd = fma((double)a.cz[k - 1], (double)(col[-k] - c) + (double)(col[k] - c), lapd);
          lapd = fma((double)a.cx[k - 1], (double)back + (double)dxf[k - 1][j], lapd);
        } else {
          lap = fmaf(a.cz[k - 1], (col[-k] - c) + (col[k] - c), lap);
          lap = fmaf(a.cx[k - 1], back + dxf[k - 1][j], lap);
        }
      }
      [[maybe_unused]] float clo = 0.f;
      if constexpr (DF) {
        const unsigned short *cll = basel + j * ROWS;
        clo = bf16_f32(cll[0]);
        lapd += (double)df_low_laplacian<ROWS>(cll, clo, c0l, a.cz, a.cx);
      }
      const int x = xs + j;
      const bool xin = x >= 0 && x < NX;                     // wave-uniform
      // r = V (L u + f);  u^{n+1} = g (2 c - g p + r)
      float r, un;
      [[maybe_unused]] unsigned short ul = 0;
      if constexpr (DF) {
        un = df_update(g[j], c, clo, pv[j], bf16_f32(pl[j]), vv[j], lapd, src[j], ul, r);
      } else {
        const float q = lap + src[j];
        un = g[j] * fmaf(q, vv[j], fmaf(c, 2.f, -(g[j] * pv[j])));
        r = vv[j] * q;
      }
      pv[j] = c;
      if constexpr (DF) pl[j] = basel[j * ROWS];
      if (!(xin && zin)) {
        un = 0.f;
        ul = 0;
      }
      [[maybe_unused]] float rs = r;
      if constexpr (FS) {
        if (z <= a.fs) {                                     // at and above the free surface
          un = rs = 0.f;
          ul = 0;
        }
      }
      const bool own = xin && x >= x0 && x < x0 + TX;        // wave-uniform
      st_f(a.out[st] + soff, keep && own ? FB : 0u, un, vz_st, x * CB);
      if constexpr (DF)
        st16(rsrc(a.lo_out[st] + soff, keep && own ? FB / 2 : 0u), ul, vz16_st, x * (CB / 2));
      if constexpr (T2) st_f(a.t2[st] + (long)s * a.t2_sstride, own ? FB : 0u, rs, vz_st, x * CB);
      if (st + 1 < kT) {
        float ut = un;
        [[maybe_unused]] unsigned short ult = ul;
        if constexpr (FS) {
          // rows fs-4 .. fs-1 of the tile: the negated mirror row 2 fs - z,
          // held by lane 2 (fs - z0 + 12) - lane of this wavefront whenever a
          // valid row reads them
          if (fs_near) {                                     // workgroup-uniform
            const int ln = ((2 * (a.fs - z0 + kHalo4) - lane) & 63) << 2;
            const float m = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(ln, __builtin_bit_cast(int, un)));
            [[maybe_unused]] int ml = 0;
            if constexpr (DF) ml = __builtin_amdgcn_ds_bpermute(ln, (int)ul);
            if (fs_mirrored(z, a.fs)) {
              ut = -m;
              if constexpr (DF) ult = (unsigned short)(ml ^ 0x8000);
            }
          }
        }
        nxt[cl + j][lz] = ut;
        if constexpr (DF) lnxt[cl + j][lz] = ult;
      }
    }
  };
  step(std::integral_constant<int, 0>{});
  if (a.steps < 2) return;
  step(std::integral_constant<int, 1>{});
  if (a.steps < 3) return;
  step(std::integral_constant<int, 2>{});
  if (a.steps < 4) return;
  step(std::integral_constant<int, 3>{});
}

template <int TX>
static hipError_t launch_step4_tx(Step4Args p, int mode, hipStream_t st) {
  const long total = (long)p.ntz * p.ntx * p.nshots;
  if (total + 8 >= (1L << 20)) return hipErrorInvalidValue;  // (choose_steps takes two steps there)
  p.by_ntz = FastDiv(p.ntz);
  p.by_ntx = FastDiv(p.ntx);
  const dim3 grid((unsigned)((total + 7) / 8 * 8));
  if (p.fs >= 0) mode |= kModeFS;
  switch (mode) {
#define FW_STEP4_MODE(M)                                               \
  case M: k_step4<TX, M><<<grid, 64 * kWaves4, 0, st>>>(p); break;     \
  case M | kModeFS: k_step4<TX, M | kModeFS><<<grid, 64 * kWaves4, 0, st>>>(p); break;
    FW_STEP4_MODE(kModePlain)
    FW_STEP4_MODE(kModeT2)
    FW_STEP4_MODE(kModeDsrc)
    FW_STEP4_MODE(kModeT2 | kModeDsrc)
    FW_STEP4_MODE(kModeNu)
    FW_STEP4_MODE(kModeDF)
    FW_STEP4_MODE(kModeT2 | kModeDF)
    FW_STEP4_MODE(kModeDsrc | kModeDF)
#undef FW_STEP4_MODE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_step4(const Step4Args &p, int tile_x, int mode, hipStream_t st) {
  if (p.steps < 1 || p.steps > kMaxSteps) return hipErrorInvalidValue;
  // a dense source or point sources, never both and never neither
  if ((mode & (kModeDsrc | kModeNu)) ? (p.inj.ptr || !p.ds[0]) : !p.inj.ptr) return hipErrorInvalidValue;
  switch (tile_x) {
    case 8: return launch_step4_tx<8>(p, mode, st);
    case 16: return launch_step4_tx<16>(p, mode, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fw
