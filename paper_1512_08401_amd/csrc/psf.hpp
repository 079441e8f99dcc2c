// Device view of a Gaussian PSF field (see psf.hip for the formula).
#pragma once

#include "common.hpp"

namespace wdb {

struct PsfDev {
  int n = 0;
  int R = 0;            // largest integer offset reachable by any PSF of the field
  double trunc = 0.0;
  double T2 = 0.0;      // trunc * trunc
  const double* sM = nullptr;
  const double* sm = nullptr;
  const double* c = nullptr;   // cos(angle), from the host libm
  const double* s = nullptr;   // sin(angle)
  const double* Z = nullptr;   // per-source normalisation sum
};

// q of source s at offset (dy, dx); the PSF reaches the offset if q <= trunc^2.
__device__ __forceinline__ double psf_q(const PsfDev& P, int64_t s, int dy, int dx) {
#pragma clang fp contract(off)
  const double c = P.c[s], sn = P.s[s], a = P.sM[s], b = P.sm[s];
  const double fx = static_cast<double>(dx), fy = static_cast<double>(dy);
  const double t1 = fx * c + fy * sn;
  const double t2 = -fx * sn + fy * c;
  return t1 * t1 / (a * a) + t2 * t2 / (b * b);
}

// exp(-q/2) if q <= trunc^2 else 0, for source s and offset (dy, dx).
__device__ __forceinline__ double psf_unnormalised(const PsfDev& P, int64_t s, int dy, int dx) {
  const double q = psf_q(P, s, dy, dx);
  return q <= P.T2 ? exp(-0.5 * q) : 0.0;
}

// A table of all weights holds the row offsets 0 .. R (a PSF is even in the offset,
// also in its roundings).
inline size_t weight_table_bytes(int64_t n, int64_t R) {
  return static_cast<size_t>((R + 1) * (2 * R + 1) * n * n) * sizeof(double);
}

// Device memory that the table may take of `free` bytes while `kept` are still to
// be allocated: an eighth of the rest, so that other threads' allocations find what
// they would find without it, all but the largest.  1024 x 1024 at radius 18 (sigma 6)
// takes 5.9 GB; without a table that build takes 12.7 s, with it 2.6 s.
inline size_t weight_table_room(size_t free, size_t kept) { return free > kept ? (free - kept) / 8 : 0; }

// Owns the uploaded field.
struct PsfField {
  int n = 0, R = 0;
  double smin = 0.0;    // least sigma
  double trunc = 0.0;
  DevBuf<double> sM, sm, cs, sn_, Z;
  ~PsfField();
  void upload(const wdb_psf_field* f, hipStream_t s);
  PsfDev dev() const;
};

}  // namespace wdb
