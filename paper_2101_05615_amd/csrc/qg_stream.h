// How the streaming kernels split their work, on the host as on the device.
#ifndef QG_STREAM_H
#define QG_STREAM_H

#ifdef __HIPCC__
#define QG_STREAM_FN static inline __host__ __device__
#else
#define QG_STREAM_FN static inline
#endif

// The build of a streaming kernel: waves of a workgroup, k blocks that a wave requests at once, fragment columns per wave.  kb: k blocks
// of a slice; sb: super-blocks of `rows` rows x 32 columns, slices counted; split: 4-bit weights.  Measured on some 150 shapes
// (M 1 .. 64, N and K 512 .. 8192, graph replays, every build on each):
//  - up to 16 k blocks four waves, up to 32 eight: one batch each, and the fewer waves there are to start and to add up the better
//    (7 x 1408 x 891: sixteen waves 4.5 us, eight 3.65; 1 x 576 x 960 3.5 and, four, 3.0);
//  - up to 64 sixteen waves (16 x 4096 x 4096: 5.2 against 6.2 with eight), beyond that eight again, whose batches follow each
//    other without a gap (1 x 704 x 5888 4.0 against 4.5); with 4-bit weights, half the bytes per batch, sixteen throughout;
//  - more workgroups of 16 columns than CUs: two fragment columns per wave (13 x 6400 x 3392 6.3 us; sixteen waves of one 8.2).
//    With 4-bit weights and a long K sixteen waves do that too (16 x 8192 x 8192 with 0.5 % of outliers 10.2 against 12.2).  At most
//    four rows and a long K, hardly any activations to share: four waves of one column again (3 x 4736 x 6848 8.4 us against 8.9,
//    2 x 7512 x 7936 11.1 against 12.3);
//  - 4-bit weights on more than 256 super-blocks: a wave's scatter of two columns in turn is what the workgroups of a CU wait for, so one
//    column again, and four waves, whose regions leave room for more workgroups per CU, most of all with batches of two.  460 shapes of M
//    1 .. 512: 16 rows 0.64 to 0.96 of the time of two columns with batches of four (7 x 8352 x 2240 with 0.5 %: 6.7 us, 4.8 so), from 513
//    on 0.74 to 0.98 of that with batches of two; 32 rows 0.71 to 0.96 of eight waves, which had taken 0.73 to 1.08 of two columns; 64 rows
//    only up to 8 k blocks (0.79 to 0.98; from 9 to 16 0.93 to 1.16).  Up to 256 super-blocks all of these lose.  (The offsets of a wave's batches lie one per lane,
//    the last one's end included: at most 63 batches, so batches of two end at 256 k blocks, 32 of them per wave.)
//    65 to 96 k blocks on 128 super-blocks and less: the second batch of sixteen waves would be half empty, eight take three (0.94 to
//    0.96, with more than 1 % of outliers 1.03 to 1.05; 9 x 1600 x 6144 4.7 us, 4.1).
struct qg_stream_build {
  int waves, batch, columns;
};
static inline qg_stream_build qg_stream_build_of(int rows, int kb, long long sb, int M, bool split) {
  const bool wide = sb > 128;
  if (rows == 16) {
    if ((kb <= 16 && !(split && sb > 512)) || (!split && wide && kb > 64 && M <= 4)) return {4, 4, 1};
    if (split && sb > 256) return sb > 512 && kb <= 256 ? qg_stream_build{4, 2, 1} : qg_stream_build{4, 4, 1};
    if (wide) return split && kb > 36 ? qg_stream_build{16, 4, 2} : qg_stream_build{8, 4, 2};
    return kb > 32 && (kb <= 64 || (split && kb > 96)) ? qg_stream_build{16, 4, 1} : qg_stream_build{8, 4, 1};
  }
  if (rows == 32) {
    if (split && sb > 256 && kb <= 256) return {4, 2, 1};
    if (wide) return split || kb <= 32 ? qg_stream_build{8, 4, 2} : qg_stream_build{4, 4, 2};
    if (kb <= 32) return {8, 4, 1};
    return split || kb > 64 ? qg_stream_build{16, 2, 1} : qg_stream_build{16, 4, 1};
  }
  if (split && sb > 256 && kb <= 8) return {4, 2, 1};
  return {8, 2, wide ? 2 : 1};
}

// Whether a 16-row kernel on 8-bit weights (and bytes of A) takes the build without the code for a K that cuts a batch: kb k blocks of a
// slice, K a whole number of them, every wave with whole batches.
static inline bool qg_stream_whole(const qg_stream_build& f, int kb, int K) {
  const int round = f.waves * f.batch;  // (a power of two)
  return K % 64 == 0 && (kb == round || (f.waves == 8 && f.columns == 2 && (kb & (round - 1)) == 0));
}

// Of those, two columns per wave with 8192 or more of K and 64 M weights (rows counted, 16 at a time) or more take four waves, batches of
// eight k blocks and activations requested at the start of a batch: what is streamed comes from HBM, and it does so faster to fewer waves
// with longer requests (16 x 8192 x 16384 28.4 us with eight, 25.2 so; 40 x 4096 x 16384 28.2 and 24.1; 16 x 8192 x 8192, weights from HBM,
// 16.0 and 15.0).  Below either bound eight are the faster: 12 x 5120 x 10240 10.4 and 11.4 us, 33 x 8192 x 4096 11.7 and 11.9.
static inline bool qg_stream_far(const qg_stream_build& f, int kb, long long sb) { return f.columns == 2 && kb >= 128 && kb * sb >= 32768; }

// The K slice that wave `wave` of workgroup `block` takes.  Workgroups go round-robin over the 8 XCDs; all workgroups of an XCD read all of
// A, and those that start on different slices request different lines of it.  Turned by `block` alone eight waves start on one slice in all
// workgroups of an XCD (block / 8 adds the turn there: 7 x 4544 x 6144 7.5 us, 6.9 so, 16 x 8192 x 8192 12.5 and 12.1, 175 shapes with more
// than 4096 columns and K from 4096 on 0.98), sixteen on two.  Those and four stay with `block` alone: sixteen make one batch each, K
// up to 4096, and every step before the first request counts (1.008 with the other, 16 x 4096 x 4096 4.55 and 4.68); four serve short K,
// where a k block's wave is best the same in the workgroups of a CU (K up to 64 1.01 to 1.09, fp32 rows up to 1.27: 123 x 640 x 16 3.3 us
// and 3.8).
QG_STREAM_FN int qg_stream_slice(int wave, unsigned block, int waves) {
  return (int)((wave + block + (waves == 8 ? block >> 3 : 0u)) % waves);
}

#endif
