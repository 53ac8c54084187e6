// Which 16-channel tiles of a 240-wide layer the wavefronts of a workgroup
// work on (fit_middle_kernel).  Plain constexpr code: it compiles on the host
// alone, where the bounds are checked.
#pragma once

constexpr int kFw = 240, kFt = kFw / 16;   // width, and its tiles

// Wavefront `wave` of `nw` owns the tiles wave, wave + nw, ... below kFt.
constexpr bool fit_owns(int wave, int nw, int u) { return wave + nw * u < kFt; }

// The u-th tile a wavefront works on: its own, or an existing one whose
// results nothing keeps (so that every wavefront reaches every barrier).
constexpr int fit_tile(int wave, int nw, int u) {
  return fit_owns(wave, nw, u) ? wave + nw * u : (wave < kFt ? wave : kFt - 1);
}

// every tile exists, and each is owned exactly once
constexpr bool fit_tiles_ok(int nw) {
  int owners[kFt] = {};
  for (int wave = 0; wave < nw; ++wave) {
    for (int u = 0; u < (kFt + nw - 1) / nw; ++u) {
      const int t = fit_tile(wave, nw, u);
      if (t < 0 || t >= kFt) return false;
      owners[t] += fit_owns(wave, nw, u) ? 1 : 0;
    }
  }
  for (int t = 0; t < kFt; ++t)
    if (owners[t] != 1) return false;
  return true;
}
