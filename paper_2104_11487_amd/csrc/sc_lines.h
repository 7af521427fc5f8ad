// Output lines on which a translated step recomputes (host and device; no HIP
// types, so the host tests compile it as plain C++).
#pragma once

#ifdef __HIPCC__
#define SC_HD __host__ __device__ __forceinline__
#else
#define SC_HD inline
#endif

namespace sc {

// Output line i (row or column) is "exposed" under a translation d of the
// input (a multiple of the stride s) when its source line i - d/s is outside
// the output grid, or when a tap p = i*s - pad + kh leaves the frame while
// p - d lies inside it: convolution and translation do not commute there.
SC_HD bool line_exposed(int i, int n_out, int n_in, int k, int s, int pad, int d) {
  if (d == 0) return false;
  const int src = i - d / s;
  if (src < 0 || src >= n_out) return true;
  for (int kh = 0; kh < k; ++kh) {
    const int q = i * s - pad + kh;
    if (q - d >= 0 && q - d < n_in && (q < 0 || q >= n_in)) return true;
  }
  return false;
}

// The exposed lines are a prefix [0, lo) and a suffix [hi, n_out). For d > 0
// the source leaves the grid on the first d/s lines, and only taps past the
// far edge can have their translated source inside; the taps of a line are
// consecutive and its first one lies inside the far edge (pad < k), so a line
// has such a tap exactly when its last one is past the edge. d < 0 mirrors it.
struct ExposedLines {
  int lo, hi;
};
SC_HD ExposedLines exposed_lines(int n_out, int n_in, int k, int s, int pad, int d) {
  ExposedLines r{0, n_out};
  if (d > 0) {
    const int first = n_in + pad - k + 1;  // i * s >= first: the last tap is past the frame
    r.lo = d / s;
    r.hi = first <= 0 ? 0 : (first + s - 1) / s;
  } else if (d < 0) {
    r.lo = (pad + s - 1) / s;  // i * s < pad: the first tap is before the frame
    r.hi = n_out + d / s;
  }
  if (r.lo > n_out) r.lo = n_out;
  if (r.hi > n_out) r.hi = n_out;
  if (r.hi < 0) r.hi = 0;
  return r;
}

}  // namespace sc
