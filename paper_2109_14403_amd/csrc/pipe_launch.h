// Host launchers of the FFT pipeline kernels. The kernels are templated on
// the line length; one object file per supported length instantiates them
// (pipe_inst.hip compiled with -DHOM_N=<n>), and the dispatchers below pick
// the instantiation at run time.
#pragma once
#include "common.h"

namespace hom {

// Supported transform lengths along every axis.
constexpr int kSupportedN[] = {16, 24, 32, 48, 64, 96, 128, 256};

inline bool supported_n(int n) {
  for (int v : kSupportedN)
    if (v == n) return true;
  return false;
}

// Elements per thread of the line FFT of length n (threads per line = n / M).
constexpr int plan_m(int n) {
  switch (n) {
    case 16: return 4;
    case 24: return 12;
    case 32: return 8;
    case 48: return 12;
    case 64: return 8;
    case 96: return 24;
    case 128: return 16;
    case 256: return 16;
  }
  return 0;
}

// x-pass lines per work-group. The FP32 middle pass holds the three CG
// fields of its voxels in registers, which allows fewer of its work-groups per
// CU: it takes half as many lines as the inverse pass, so more, smaller
// work-groups overlap their load and transform phases.
constexpr int x_lines(int n, bool fp64, bool mid) {
  const int nl = ((fp64 ? 64 : 128) / (n / plan_m(n))) / (mid && !fp64 ? 2 : 1);
  return nl < 1 ? 1 : nl;
}
// Launches of few lines take a quarter of that in the middle pass, so that the
// lines spread over more of the chip. Measured on increments of single cells
// (in brackets the work-groups they made before): FP64 32 x 16^2 (16) 1.12, 24^3
// (36) 1.19, 32^3 (64) 1.06, 96 x 24 x 48 (72) 1.14, 128 x 32 x 32 (128) 1.08, 48^3
// (144) 1.03 times as fast; FP32 24^3 (18) 1.06, 32^3 (64) 1.05, 96 x 24 x 48 (72)
// 1.10, but 128 x 32 x 32 (128) 0.98 and 48^3 (144) 0.99. The fixed-point scheme's
// middle pass: 16^3 1.05, 32^3 FP64 1.03, FP32 1.06, 24 x 16 x 32 FP32 1.14 (its
// separate forward and inverse passes: 16^3 0.97, left as they are).
constexpr int xmid_lines_few(int n, bool fp64) {
  return x_lines(n, fp64, true) < 4 ? 1 : x_lines(n, fp64, true) / 4;
}
constexpr int xmid_lines(int n, bool fp64, long long lines) {
  return lines < (fp64 ? 256LL : 112LL) * x_lines(n, fp64, true) ? xmid_lines_few(n, fp64) : x_lines(n, fp64, true);
}

// Schedules of the y and z passes: tile width (kx columns per work-group: 2,
// 4 or 8) and FFT plan variant (0 or 1, Plan<N, V>), packed as width + 16 V.
// The autotuner times every one on the problem's own data.
constexpr int schedule(int tile, int plan) { return tile + 16 * plan; }
constexpr int schedule_tile(int s) { return s & 15; }
constexpr int schedule_plan(int s) { return s >> 4; }
constexpr int kScheduleChoices[] = {schedule(2, 0), schedule(4, 0), schedule(8, 0),
                                    schedule(2, 1), schedule(4, 1), schedule(8, 1)};

// The plane pass holds a whole ny x nz plane of one kx, all components, in LDS
// (rows of plane_row complex values: padding spreads the rows of a y transform
// over the banks), and the twiddles of both axes.
constexpr int plane_row(int ny, int C) { return (ny + 1) * C; }
constexpr size_t plane_lds(int ny, int nz, int C, bool fp64) {
  return ((size_t)nz * plane_row(ny, C) + ny + nz) * (fp64 ? 16 : 8);
}
constexpr bool plane_fits(int ny, int nz, bool fp64) { return plane_lds(ny, nz, 6, fp64) <= 120 * 1024; }
// The plane pass puts a plane on one CU, the three separate passes spread it
// over the chip but make three trips and two more launches. Measured:
// single cells (increments of 32 x ny x nz, 17 planes on 256 CUs) in FP32 16^2
// 1.33, 24^2 1.26, 32^2 1.19, 24 x 48 1.16, 64 x 24 1.05, 96 x 16 1.11, 64 x 32
// (98 KB) 1.04 times as fast, 48^2 (113 KB) 0.93; in FP64 16^2 1.22, 24^2
// (58 KB) 1.15, 32^2 (101 KB) 0.98, 24 x 48 0.90. Batches, FP32: 8 and 64
// problems of 24^3 1.18 and 1.05, of 32^3 1.13 and 1.14, 8 and 32 of 48^3 (200
// and 800 planes) 1.12 and 1.10. So large planes need enough of them.
inline bool plane_pass(int ny, int nz, bool fp64, long long planes) {
  return plane_fits(ny, nz, fp64) &&
         (plane_lds(ny, nz, 6, fp64) <= (size_t)(fp64 ? 64 : 104) * 1024 || planes >= 128);
}

struct LaunchInfo {
  int blocks;
  int threads;
  size_t lds;
};

template <typename T, int N>
LaunchInfo xfwd_launch(const Pipe<T>& a, hipStream_t s, bool dry);
template <typename T, int N>
LaunchInfo xinv_launch(const Pipe<T>& a, hipStream_t s, bool dry);
template <typename T, int N>
LaunchInfo xmid_launch(const Pipe<T>& a, hipStream_t s, bool dry);
template <typename T, int N>
LaunchInfo xbasic_launch(const Pipe<T>& a, hipStream_t s, bool dry);
template <typename T, int N>
LaunchInfo ypass_launch(const Pipe<T>& a, int sched, int inverse, hipStream_t s, bool dry);
template <typename T, int N>
LaunchInfo zgreen_launch(const Pipe<T>& a, int sched, hipStream_t s, bool dry);
template <typename T, int N>  // N = nz; a.ny one that fits
LaunchInfo yzplane_launch(const Pipe<T>& a, hipStream_t s, bool dry);

template <typename T>
LaunchInfo run_xfwd(const Pipe<T>& a, hipStream_t s, bool dry = false);
template <typename T>
LaunchInfo run_xinv(const Pipe<T>& a, hipStream_t s, bool dry = false);
template <typename T>
LaunchInfo run_xmid(const Pipe<T>& a, hipStream_t s, bool dry = false);
template <typename T>
LaunchInfo run_xbasic(const Pipe<T>& a, hipStream_t s, bool dry = false);
template <typename T>
LaunchInfo run_ypass(const Pipe<T>& a, int sched, int inverse, hipStream_t s, bool dry = false);
template <typename T>
LaunchInfo run_zgreen(const Pipe<T>& a, int sched, hipStream_t s, bool dry = false);
template <typename T>
LaunchInfo run_yzplane(const Pipe<T>& a, hipStream_t s, bool dry = false);

}  // namespace hom
