// Exact image positions without a division per lane, on the host as on the device.
#ifndef QG_POSITION_H
#define QG_POSITION_H

#ifdef __HIPCC__
#define QG_POSITION_FN static inline __host__ __device__
#else
#define QG_POSITION_FN static inline
#endif

// Exact unsigned division by a number the host knows: q = (t + ((n - t) >> s1)) >> s2 with t the high word of m * n (Granlund
// and Montgomery, "Division by invariant integers using multiplication", 1994).  On a wave-uniform n all of it runs on the
// scalar unit; an integer division is 25 vector instructions.
struct qg_udiv {
  unsigned m, s;  // s: s1 | s2 << 8
};
static inline qg_udiv qg_make_udiv(unsigned d) {
  int l = 0;
  while ((1ull << l) < d) ++l;
  const unsigned m = (unsigned)((((1ull << l) - d) << 32) / d) + 1u;
  return {m, (unsigned)(l < 1 ? l : 1) | (unsigned)(l > 0 ? l - 1 : 0) << 8};
}
QG_POSITION_FN unsigned qg_quot(unsigned n, unsigned m, unsigned s) {
  const unsigned t = (unsigned)(((unsigned long long)m * n) >> 32);
  return (t + ((n - t) >> (s & 1))) >> (s >> 8 & 31);
}

// Row and column, inside their image, of pixel first + step of a sequence of H x W images; step is at most 31.  `first` is
// wave-uniform (a wave's first pixel), so only what follows from `step` is left to the lanes.  Every step is exact for all
// extents: from 2^23 pixels on, an fp32 quotient is not.
QG_POSITION_FN void qg_pixel_position(unsigned first, unsigned step, unsigned W, unsigned mW, unsigned sW, unsigned H, unsigned mH,
                                      unsigned sH, int* row, int* col) {
  const unsigned row0 = qg_quot(first, mW, sW);
  unsigned wo = first - row0 * W + step;
  unsigned ho = row0 - qg_quot(row0, mH, sH) * H;
  if (W > 31) {  // at most one row further
    if (wo >= W) wo -= W, ++ho;
    if (ho == H) ho = 0;
  } else {
    const unsigned rows = qg_quot(wo, mW, sW);
    wo -= rows * W;
    ho += rows;
    ho -= qg_quot(ho, mH, sH) * H;
  }
  *row = (int)ho;
  *col = (int)wo;
}

#endif
