// Host side of the C ABI declared in qgemm.h: argument checks, descriptor
// bookkeeping and kernel selection by shape.  No device allocation, no stream
// creation, no synchronisation happens here (paper Appendix A: the library works
// on caller-provided buffers and leaves parallelism to the caller).
#include <math.h>

#include <new>
#include <vector>

#include "qg_internal.h"

namespace {

inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int check_requant(const qg_requant_params* p, int N) {
  if (!p) return QG_ENULL;
  if (!p->scales) return QG_ENULL;
  if (p->a_zp < 0 || p->a_zp > 255 || p->c_zp < 0 || p->c_zp > 255) return QG_EINVAL;
  if (p->n_scales != 1 && p->n_scales != N) return QG_EINVAL;
  if (p->relu != 0 && p->relu != 1) return QG_EINVAL;
  return QG_OK;
}

// Builds the padded per-column theta_B array on the host and enqueues its upload
// into the second half of the caller's col_offsets buffer.
int upload_bzp(const int32_t* b_zp_host, int n_b_zp, int N, int N_pad, int32_t* dst_dev, hipStream_t s,
               int* has_bzp) {
  std::vector<int32_t> tmp;
  try {
    tmp.assign((size_t)N_pad, 0);
  } catch (const std::bad_alloc&) {
    return QG_ENOMEM;
  }
  int any = 0;
  for (int j = 0; j < N; ++j) {
    const int32_t z = b_zp_host[n_b_zp == 1 ? 0 : j];
    if (z < -128 || z > 127) return QG_EINVAL;
    tmp[j] = z;
    any |= (z != 0);
  }
  *has_bzp = any;
  // pageable source: the runtime stages it before returning, so tmp may die here
  if (hipMemcpyAsync(dst_dev, tmp.data(), sizeof(int32_t) * (size_t)N_pad, hipMemcpyHostToDevice, s) !=
      hipSuccess)
    return QG_ELAUNCH;
  if (hipStreamSynchronize(s) != hipSuccess) return QG_ELAUNCH;  // offline path; keeps tmp's lifetime trivially safe
  return QG_OK;
}

// ---- kernel selection by shape (paper Appendix C) --------------------------------------------
qg_dispatch_rule g_rules[QG_MAX_DISPATCH_RULES];
int g_nrules = 0;

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Built-in choice: a small cost model of every kernel, fitted to timings of the whole family over a grid of
// shapes on MI355X (256 CUs), evaluated for the shape at hand; the cheapest estimate wins.
//
// Tiled kernels.  A workgroup alone on the chip needs `lat` us per 64-deep k step (one barrier plus request
// latency) and `fix` us of launch, prologue and output pipeline.  With the chip full, each of the
// ceil(workgroups / 256) workgroups a CU has to run costs `thr` us per k step and `epi` us of output
// pipeline: a big tile moves the fewest LDS bytes per multiply (small `thr` per unit of work) but pays for
// it with few, long workgroups.  The estimate is the larger of the two regimes; a grid of at most one
// workgroup per CU is in the first by definition.
// Streaming kernels.  One workgroup per 16 columns and per row block; alone it takes fix + K * lat_k us, with
// the chip full each workgroup costs wg + K * wg_k nanoseconds; a third bound covers tall, narrow shapes.
struct tile_cost {
  int kernel, bm, bn;
  double fix, lat, thr, epi;
  double out = 0.0;  // output bytes per microsecond that the kernel sustains when K is short; 0 = never the bound
};
struct stream_cost {
  int kernel, rows;
  double fix, lat_k, wg, wg_k;
};
const tile_cost k_tile_cost[] = {
    {QG_KERNEL_TILE64, 64, 64, 3.169, 0.1296, 0.1046, 0.6015},
    {QG_KERNEL_TILE128, 128, 128, 3.401, 0.242, 0.2725, 1.102, 2.88e6},
    {QG_KERNEL_TILE128X256, 128, 256, 5.288, 0.3543, 0.4409, 2.253},
    {QG_KERNEL_TILE256, 256, 256, 7.789, 0.6867, 0.8478, 6.549},
    {QG_KERNEL_TILE64K4, 64, 64, 3.617, 0.1035, 0.1077, 2.38},
    {QG_KERNEL_TILE64K1, 64, 64, 2.714, 0.2482, 0.1361, 0.1909, 2.35e6},
    {QG_KERNEL_TILE64X32K8, 64, 32, 3.817, 0.05427, 0.0602, 2.585},
};
// (Of the streaming kernels' former builds, sixteen waves throughout: what was announced by them stays announced.)
const stream_cost k_stream_cost[] = {
    {QG_KERNEL_SKINNY16, 16, 3.826, 3.664e-06, 5.429, 0.002625},
    {QG_KERNEL_SKINNY32, 32, 3.918, 2.404e-05, 8.639, 0.0005841},
    {QG_KERNEL_SKINNY64, 64, 3.821, 0.0004905, 9.136, 0.002971},
};
// The 16-row kernel on more than 128 super-blocks of 16 rows x 32 columns with K a multiple of 2048 and dense weights, which all ran in
// a form of four waves then (that form serves large ones only now): the same formula per super-block.
const stream_cost k_stream_wide_cost = {QG_KERNEL_SKINNY16, 16, 3.191, 0.0002712, 4.302e-05, 0.001958};
// A streaming workgroup re-reads its rows of A for every 16 columns; with few columns to share them that
// traffic comes from far memory, row piece by row piece, at about this many bytes per microsecond.
const double k_stream_a_rate = 2.0e6;
const double k_stream_a_near = 1048576.0;     // bytes of A that the L2s keep
const double k_stream_a_far_rate = 1.0e7;     // bytes per microsecond, all workgroups together

double stream_estimate(const stream_cost& c, int M, int N, int K, bool dense) {
  double a_bound = 2.5 + (double)M * (double)K / k_stream_a_rate;
  const double blocks32 = (double)ceil_div(M, c.rows) * (double)ceil_div(N, 32);
  if (dense && c.kernel == QG_KERNEL_SKINNY16 && blocks32 > 128.0 && K % 2048 == 0) {
    const stream_cost& w = k_stream_wide_cost;
    return fmax(fmax(w.fix + K * w.lat_k, a_bound), 2.5 + blocks32 * (w.wg + K * w.wg_k) * 1e-3);
  }
  const double wgs = 2.0 * blocks32;
  // an A too large to stay in the L2s is fetched from far memory once per 16 columns
  if ((double)M * (double)K > k_stream_a_near)
    a_bound = fmax(a_bound, 2.5 + (double)M * (double)K * (double)ceil_div(N, 16) / k_stream_a_far_rate);
  const double alone = fmax(c.fix + K * c.lat_k, a_bound);
  if (wgs <= 256.0) return alone;  // at most one workgroup per CU: each runs as if alone
  return fmax(alone, 2.5 + wgs * (c.wg + K * c.wg_k) * 1e-3);
}

double tile_estimate(const tile_cost& c, int M, int N, int K) {
  const double kt = (double)ceil_div(K, 64);
  const double wgs = (double)ceil_div(M, c.bm) * (double)ceil_div(N, c.bn);
  const double alone = c.fix + kt * c.lat;
  if (wgs <= 256.0) return alone;
  double us = fmax(alone, 2.5 + ceil(wgs / 256.0) * (kt * c.thr + c.epi));
  // many rows and a K of one or two tiles (the 1 x 1 layers of a convolutional network as GEMMs): little but output,
  // at a rate measured on 30 such shapes (without this bound the 64 x 64 tile was chosen for 100352 x 256 x 64,
  // 1.15x behind the 128 x 128 tile)
  if (c.out > 0.0) us = fmax(us, 2.5 + (double)M * (double)N / c.out);
  return us;
}

// What the queries about K splits and workspaces, calls that ask for a split and calls that bring a workspace for one go by, and whether
// fp32 activations without a workspace are served: one answer for a shape, whatever the alignment of the operands.
int builtin_select(int M, int N, int K) {
  int best = QG_KERNEL_TILE64;
  double best_us = 1e300;
  for (const stream_cost& c : k_stream_cost) {
    const long long blocks = ceil_div(M, c.rows);
    if (blocks > 65535) continue;
    const double us = stream_estimate(c, M, N, K, true);
    if (us < best_us) best_us = us, best = c.kernel;
  }
  for (const tile_cost& c : k_tile_cost) {
    const double us = tile_estimate(c, M, N, K);
    if (us < best_us) best_us = us, best = c.kernel;
  }
  return best;
}

// All other calls: the same idea with the terms that decide close races, fitted anew.
//   tile, at most 256 workgroups   us = fix + kt * (lat * (1 + tall * M / (M + N)) + crowd * wgs / 256)     kt = ceil(K / 64)
//   beyond                         the larger of that and 2.5 + rounds * epi + kt * thr * (rounds - fill * (rounds - wgs / 256)),
//                                  rounds = ceil(wgs / 256): a round that does not fill the chip runs faster
//   streaming                      us = fix + K / 1024 * (lat + crowd * wgs / 256) + blocks * block + n * batch + what is fetched, waves
//                                  and blocks those of the build; more than 256 workgroups: the larger of that times (1 + second) and
//                                  `round` per further 256, and 2.5 + wgs * (wg + K * wg_k) ns
// and far more per megabyte of A beyond four.  Fitted to graph-replay times of all kernels on 46417 drawn shapes (M 1 .. 65536, N 8 ..
// 8192, K 16 .. 16384, rows of A and C at all alignments, the three kinds of results, with and without zero points) and 5600 round
// ones, three sets of buffers in turn: first the times, then the loss of the choice.  Over 7600 other drawn shapes the choice is 1.0034
// of the best kernel in the geometric mean, 1.32 at worst, 178 of them by more than 5 %; over 1400 other round ones 1.0030, 1.20 and
// 31.  The prices above: 1.050 and 1.026; a fit to ordinary shapes alone: 1.020 and 1.026, 2.5 at worst (tall shapes of few columns and
// a long K: 827 x 17 x 15685 25.1 us, 10.4 on the 16-row kernel).
// The streaming kernels' prices are newer: fitted to 39000 shapes, columns up to 32768 and K of whole 256, 1024 and 2048 among them, with
// those kernels as they are now (times scaled to the price of the best tiled kernel on each, then the loss of the choice; no choice is
// held).  Over 3000 others the choice is 1.0048 of the best kernel, 104 by more than 5 %; the former prices, which had two choices held,
// 1.0151 and 306, and on up to 24 rows with 2048 columns and more 1.033, now 1.0062 (9 x 6208 x 6752 10.9 us, 8.9 now; 14 x 5632 x 3648
// 7.1, 5.8).  On 1200 large products 1.0094, by the prices of the tiled kernels.
struct tile_price {
  int kernel, bm, bn;
  double fix, lat, crowd, thr, fill, epi, out;         // out: megabytes of output per microsecond
  double f32_fix, f32_epi, rag_fix, rag_epi;           // fp32 results; u8 results whose rows start off 16 bytes
  double tail_fix, tail_epi;                           // K off 16: the bytes past it are masked one by one
  double fix4, fix1, lat4, lat1, thr4, thr1;           // rows of A at multiples of 4 bytes, at any: additions and factors
  double i32_fix, i32_epi, tall, far;                  // int32 results; fewer workgroups share a row of A; megabytes of A beyond 4
  double left_fix, left_epi;                           // K off 64: the last tile is staged through registers
  double bzp_fix, bzp_lat, bzp_thr;                    // weight zero points: the row sums; additions to lat and thr as factors
  double b_far, b_near, half;                          // us per megabyte of B beyond b_near; last column of tiles at most half full: adds to lat
};
struct stream_price {
  int kernel, rows;
  double fix, fix8, fix16;                             // fix8, fix16: added for eight and sixteen waves
  double lat, crowd;                                   // per 1024 of K; on a full chip
  double block, batch;                                 // per k block of a wave; per batch that it requests after its first
  double second, wg, wg_k;                             // more than 256 workgroups: share on top; ns per workgroup, per 1 of K
  double bzp_fix, bzp_lat, tail_fix;                   // weight zero points; K off 16
  double fix4, fix1, lat4, lat1, wg_k4, wg_k1;         // rows of A at multiples of 4 bytes, at any: additions and factors
  double f32_fix, f32_wg, i32_fix, i32_wg;
  double a_far, far;                                   // tens of megabytes of A per us, once per column block from beyond the L2s; beyond 4
  double fetch, near;                                  // us per megabyte that the XCDs fetch beyond so many
  double round;                                        // per round of 256 workgroups after the first
  double b_far, b_near;                                // us per megabyte of B beyond b_near
  double whole;                                        // so much less where the batches of all waves are whole
  double more_second, more_wg_k;                       // more than one row block, which share the weights: second; factor of wg_k
};
// The second of QG_KERNEL_TILE128 is the 128 x 64 form, which runs on at most one workgroup per CU (its terms beyond are zero).
const tile_price k_tile_price[] = {
    {QG_KERNEL_TILE64K1, 64, 64, 2.379, 0.2932, 0.01648, 0.1083, 0.3038, 0.2923, 5.958, 0, 0.09458, 0.09551, 0.08843,
     0.4098, 0.0001485, 0.1085, 0.2234, 0.9467, 0.7933, 1.137, 1.339, 1.536, 3.088, 0, 0.07322, 0.281, 0.05757, 0.1985,
     0.1236, 0.1061, 0.09257, 2.034, 0.1429},
    {QG_KERNEL_TILE64, 64, 64, 3.18, 0.1188, 0.0262, 0.1003, 0.2297, 0.6596, 4.039, 0, 0.1417, 0.1046, 0.1366, 0.3663,
     0.09615, 0.09498, 0.0814, 0.908, 1.045, 1.087, 1.341, 1.607, 2.876, 0.03544, 0.05423, 0.3726, 0.1756, 0.1533,
     0.1031, 0.1138, 0.03702, 5.898, 0.04424},
    {QG_KERNEL_TILE64K4, 64, 64, 3.925, 0.08141, 0.01436, 0.1072, 0.3085, 1.888, 3, 0.1155, 0.2087, 0.1261, 0.1871,
     0.395, 0.02942, 0.000062, 0.06287, 1.051, 1.419, 1.07, 1.339, 1.61, 3.744, 0.03794, 0.07046, 0.355, 0.515, 0.2,
     0.1045, 0.1487, 0.01903, 0.005161, 0.03733},
    {QG_KERNEL_TILE64X32K8, 64, 32, 3.889, 0.05234, 0.0141, 0.05647, 0.1724, 2.277, 3, 0.1677, 0.1599, 0.1178, 0.5721,
     0.3305, 0.2734, 0.0001932, 0.1679, 1.085, 1.86, 1.402, 1.57, 1.172, 2.852, 0.008428, 0.06507, 0.6046, 0.3201,
     0.2513, 0.06846, 0.2169, 0.358, 83.9, 0.01019},
    {QG_KERNEL_TILE128, 128, 128, 4.588, 0.1417, 0.1085, 0.281, 0.4045, 1.211, 4.552, 0.06927, 0.6241, 0.4908, 0.3061,
     0.1743, 0.01932, 0.1741, 0, 1.194, 1.42, 1.104, 1.299, 10.24, 11.93, 0.01551, 0.05237, 0.7058, 0.1994, 0.000086,
     0.1634, 0.09938, 0.04505, 10.17, 0.1441},
    {QG_KERNEL_TILE128, 128, 64, 5.169, 0.08882, 0.04409, 0, 0, 0, 3, 0.654, 0, 0.4652, 0, 0.5053, 0, 0.6046, 1.463,
     1.016, 1.37, 0, 0, 6.708, 0, 0.08092, 0.05976, 0.9807, 0, 0.000098, 0.1067, 0.01832, 0.01736, 14.16, 0.04551},
    {QG_KERNEL_TILE128X256, 128, 256, 6.811, 0.1843, 0.1932, 0.4171, 0.2032, 2.807, 5.18, 0.3315, 0.4456, 0.626, 0.5827,
     0.4845, 0.03141, 0.6825, 0.8138, 1.077, 1.314, 1.101, 1.184, 22.27, 23.48, 0.0352, 0.06443, 0.2875, 0.3988, 0.1165,
     0.201, 0.08051, 0.06708, 16.31, 0.3304},
    {QG_KERNEL_TILE256, 256, 256, 15.64, 0.2597, 0.4748, 0.7312, 0.401, 10.36, 3.674, 0.00005, 0.0004028, 0.4451, 1.441,
     1.151, 0.003431, 2.957, 0.0002237, 0.8557, 1.931, 1.107, 1.306, 46.77, 53.72, 0.000361, 0, 0.0003799, 2.048,
     0.0006701, 0.1854, 0.1629, 0.0001407, 11.17, 0.1874},
};
// (in pairs: up to 128 super-blocks of rows x 32 columns, where the terms for more workgroups than CUs are left out, and more; then the
// other builds and depths beyond 128: 16 rows, four waves of one column, for up to four rows and a long K and for up to 16 k blocks; 32
// rows, up to 32 k blocks; 16 rows, up to 32; 16 rows, four waves with batches of eight.  That one is fitted to 230 drawn
// shapes of its range, up to 400 M weights: 1.028 of the best kernel, 1.033 by the second row)
const stream_price k_stream_price[] = {
    {QG_KERNEL_SKINNY16, 16, 2.983, 0.02822, 0.4741, 0.05277, 0.09842, 5.28e-05, 0.4466, 0, 0, 0, 3.543e-05, 0.0001109,
     2.635e-05, 0.04294, 0.09123, 1.033, 1.5, 0, 0, 0, 0, 0, 0, 0.9646, 0.1252, 0.04834, 3.62, 0, 0.0002, 70, 0.3493,
     0, 0},
    {QG_KERNEL_SKINNY16, 16, 0.1835, 3.345, 0.5, 0.01965, 0.001042, 0.0001344, 0.5185, 0.007127, 0.1403, 0.002334,
     0.009597, 0.06298, 6.566e-05, 0.126, 0.02872, 0.9085, 1.581, 0.9083, 1.414, 0.0007144, 0.5192, 0.03076, 1.939,
     1.5, 0.01412, 0.0865, 4.574, 1.375, 0.07699, 54.84, 0.1727, 0.1886, 1.417},
    {QG_KERNEL_SKINNY32, 32, 3.253, 0.1344, 0.6943, 0.05584, 0.01053, 4.352e-05, 0.513, 0, 0, 0, 0.00434, 0.03572,
     0.07619, 0.05571, 0.4104, 1.079, 1.805, 0, 0, 0.0007931, 0, 2.402e-05, 0, 0.8106, 0.1573, 0.06216, 0.004036, 0,
     0.0002, 70, 0, 0, 0},
    {QG_KERNEL_SKINNY32, 32, 3.322, 0.0002, 0.5, 0.02931, 0.1067, 0.0002637, 0.2814, 0.2265, 0.02392, 0.0009932,
     0.001088, 0.108, 0.01154, 0.01654, 0.1137, 1.037, 1.971, 1.695, 3.052, 0.1929, 0.05645, 0.03491, 0.0003043,
     0.9501, 0.001606, 0.07357, 0.1386, 1.427, 0.03674, 2.958, 0, 0.362, 1.985},
    {QG_KERNEL_SKINNY64, 64, 3.235, 0.1673, 0.5, 0.1411, 0.1045, 0.0001145, 0.3719, 0, 0, 0, 0.005093, 0.05883, 0.1144,
     0.1041, 0.2901, 1.201, 2.144, 0, 0, 0.163, 0, 0.4691, 0, 2.087, 0.2004, 0.06998, 0.0004859, 0, 0.0002, 70, 0, 0,
     0},
    {QG_KERNEL_SKINNY64, 64, 3.521, 0.1821, 0.5, 0.1256, 0.005196, 7.668e-05, 0.4534, 0.5234, 6.514, 0.003999, 0.1165,
     0.1458, 0.2133, 0.06736, 0.4308, 1.16, 1.977, 1.394, 1.881, 0.122, 0.1533, 0.0002338, 0.2097, 1.912, 0.000961,
     0.1102, 0.06496, 2.123, 0.0002, 140.4, 0, 0.2827, 1.416},
    {QG_KERNEL_SKINNY16, 16, 1.903, 2.606, 0.5, 0.1963, 0.07251, 0.0001901, 0.1182, 0.07707, 0.4461, 0.001301, 0.0198,
     0.1311, 0.01446, 0.003134, 0.1067, 1.052, 1.128, 0.9856, 0.9931, 0.005627, 0.03856, 0.04532, 0.005549, 1.5,
     0.007077, 0.06172, 1.077, 1.26, 0.08207, 73.4, 0.01, 0.09177, 1},
    {QG_KERNEL_SKINNY16, 16, 1.344, 2.896, 0.5, 5.368e-05, 2.095e-05, 0, 0.006053, 0.04129, 1.606, 6.097e-05, 0.09463,
     0.003243, 0.04371, 0.0541, 0.4061, 0.02498, 0.02293, 6.854, 11.76, 0.0007712, 0.1865, 0, 0, 1.5, 0.3297, 0.09574,
     0.1461, 0.6666, 0.0002, 70, 0.6227, 0.2078, 0.2314},
    {QG_KERNEL_SKINNY32, 32, 3.676, 0.0002025, 0.5, 0.003235, 0.003171, 3.276e-05, 0.2263, 0.1643, 6.496, 0.006098,
     0.008458, 0.03281, 0.1052, 0.09962, 0.243, 0.00297, 38.2, 1.109, 1.27, 0.04818, 0.05044, 0.1093, 3.298, 1.008,
     0.02535, 0.07889, 0.06179, 2.329, 0.0002, 70, 0, 0.1023, 0.08342},
    {QG_KERNEL_SKINNY16, 16, 0.1639, 2.988, 0.5, 0.1175, 0.06546, 0.0001377, 0.3826, 0.0003874, 1.832, 0.001001,
     0.0195, 0.07932, 0.08213, 0.009258, 0.1466, 1.15, 1.628, 0.9652, 1.059, 0.005616, 0.6934, 0.009526, 0.0002023,
     1.5, 0, 0.1091, 6.622, 1.005, 0.03082, 68.34, 0.007549, 0.08187, 0.5645},
    {QG_KERNEL_SKINNY16, 16, 0.1835, 2.442, 0.5, 0.01965, 0.001042, 0.02858, 0.3986, 0.2733, 2.584, 0.002622, 0.009597,
     0.4563, 6.566e-05, 0.126, 0.02872, 0.8811, 0.0008504, 0.7344, 1.249, 0.0007144, 0.5192, 0.03076, 1.939, 1.5,
     0.0008048, 0.08125, 18.52, 2.52, 0.04573, 10.04, 0.1727, 0.423, 1.235},
};

enum out_kind { OUT_U8, OUT_U8_RAGGED, OUT_F32, OUT_I32 };  // RAGGED: rows of C off 16 bytes
struct call_form {
  int a_align;  // 16: base and rows of A at multiples of 16 bytes, 4: of 4 bytes, 1: others
  out_kind out;
  bool bzp;     // weight zero points
};

// (plain comparisons and integer rounds: the library functions are calls on the baseline target, and every call of the GEMM comes here)
inline double larger(double a, double b) { return a > b ? a : b; }
inline long long tiles_of(int M, int N, int bm, int bn) { return (long long)ceil_div(M, bm) * ceil_div(N, bn); }
inline double rounds_of(long long wgs) { return (double)((wgs + 255) / 256); }
inline double share_of_chip(long long wgs) { return wgs < 256 ? (double)wgs / 256.0 : 1.0; }

double tile_price_us(const tile_price& c, int M, int N, int K, const call_form& f) {
  const double kt = (double)ceil_div(K, 64);
  const long long wgs = tiles_of(M, N, c.bm, c.bn);
  const int a = f.a_align == 16 ? 0 : f.a_align == 4 ? 1 : 2;
  const bool tail = K % 16 != 0, left = K % 64 != 0, wide = f.out >= OUT_F32;
  const double out_fix[] = {0.0, c.rag_fix, c.f32_fix, c.i32_fix}, out_epi[] = {0.0, c.rag_epi, c.f32_epi, c.i32_epi};
  const double a_fix[] = {0.0, c.fix4, c.fix1}, a_lat[] = {1.0, c.lat4, c.lat1}, a_thr[] = {1.0, c.thr4, c.thr1};
  const double fix = c.fix + out_fix[f.out] + a_fix[a] + (tail ? c.tail_fix : 0.0) + (left ? c.left_fix : 0.0) + (f.bzp ? c.bzp_fix : 0.0);
  const double lat = c.lat * a_lat[a] * (f.bzp ? 1.0 + c.bzp_lat : 1.0) * (1.0 + c.tall * M / ((double)M + N)) *
                     (N % c.bn != 0 && N % c.bn <= c.bn / 2 ? 1.0 + c.half : 1.0);
  double us = larger(fix + kt * (lat + c.crowd * share_of_chip(wgs)), 2.5 + (double)M * (double)N * (wide ? 4.0 : 1.0) / (c.out * 1e6));
  if (wgs > 256) {
    // (what 4-byte results cost goes by the columns there are: 53310 x 12 x 256 to int32 10.8 us on the 64-row kernel, 6.9 on 64 x 64 tiles)
    const double epi = c.epi + out_epi[f.out] * (c.bn <= 64 && N < c.bn ? (double)N / c.bn : 1.0) + (tail ? c.tail_epi : 0.0) + (left ? c.left_epi : 0.0);
    const double rounds = rounds_of(wgs), steps = rounds + c.fill * ((double)wgs / 256.0 - rounds);
    us = larger(us, 2.5 + rounds * epi + steps * kt * c.thr * a_thr[a] * (f.bzp ? 1.0 + c.bzp_thr : 1.0));
  }
  return us + c.far * larger((double)M * K * 1e-6 - 4.0, 0.0) + c.b_far * larger((double)K * N * 1e-6 - c.b_near, 0.0);
}

// what the builds of the streaming kernels share: extents of a launch (powers of two throughout: shifts, no divisions)
struct stream_shape {
  int kb, per, batches;  // k blocks, of a wave, batches after a wave's first
  int row_blocks, columns;
  long long sb, wgs;     // super-blocks of rows x 32 columns, workgroups
  qg_stream_build f;
  bool far;              // four waves, batches of eight (8-bit weights and rows of bytes)
};
inline int ceil_shift(int a, int s) { return ((a - 1) >> s) + 1; }  // a >= 1
stream_shape shape_of(int rows, int M, int N, int K, bool split = false) {
  stream_shape s;
  s.kb = ceil_shift(K, 6);
  s.row_blocks = ceil_shift(M, __builtin_ctz(rows));
  s.sb = (long long)s.row_blocks * ceil_shift(N, 5);
  s.f = qg_stream_build_of(rows, s.kb, s.sb, M, split);
  s.far = rows == 16 && !split && qg_stream_whole(s.f, s.kb, K) && qg_stream_far(s.f, s.kb, s.sb);
  const int w = __builtin_ctz(s.f.waves);
  s.per = split ? 2 * ceil_shift(s.kb, w + 1) : ceil_shift(s.kb, w);
  s.batches = ceil_shift(s.per, __builtin_ctz(s.f.batch)) - 1;
  s.columns = ceil_shift(N, s.f.columns == 2 ? 5 : 4);
  s.wgs = s.f.columns == 2 ? s.sb : 2 * s.sb;
  return s;
}

// megabytes that the XCDs fetch, an operand counted once for each: column block j of row block i runs on XCD (i * columns + j) % 8
double fetched_mb(const stream_shape& s, int M, int N, int K) {
  const int spread = s.columns % 8 ? 8 >> __builtin_ctz(s.columns) : 1;
  return ((double)(s.row_blocks < spread ? s.row_blocks : spread) * N + (double)(s.columns < 8 ? s.columns : 8) * M) * K * 1e-6;
}

double stream_price_us(const stream_price& c, const stream_shape& s, int M, int N, int K, const call_form& f) {
  // (with a quarter of the rows or less a quarter of them is requested, and their alignment hardly counts)
  const int a = f.a_align == 16 || 4 * M <= c.rows ? 0 : f.a_align == 4 ? 1 : 2;
  const double out_fix[] = {0.0, 0.0, c.f32_fix, c.i32_fix}, out_wg[] = {0.0, 0.0, c.f32_wg, c.i32_wg};
  const double a_fix[] = {0.0, c.fix4, c.fix1}, a_lat[] = {1.0, c.lat4, c.lat1}, a_wg_k[] = {1.0, c.wg_k4, c.wg_k1};
  const double bzp = f.bzp ? 1.0 + c.bzp_lat : 1.0;
  const double fix = c.fix + (s.f.waves == 8 ? c.fix8 : s.f.waves == 16 ? c.fix16 : 0.0) + out_fix[f.out] + a_fix[a] +
                     (K % 16 != 0 ? c.tail_fix : 0.0) + (f.bzp ? c.bzp_fix : 0.0) - (c.rows == 16 && qg_stream_whole(s.f, s.kb, K) ? c.whole : 0.0);
  double us = fix + (K / 1024.0 * (c.lat + c.crowd * share_of_chip(s.wgs)) + s.per * c.block + s.batches * c.batch) * bzp * a_lat[a] +
              c.fetch * larger(fetched_mb(s, M, N, K) - c.near, 0.0);
  if (s.wgs > 256)
    us = larger(us * (1.0 + (M > c.rows ? c.more_second : c.second)) + (rounds_of(s.wgs) - 1.0) * c.round,
                2.5 + (double)s.wgs * (c.wg + out_wg[f.out] + K * c.wg_k * (M > c.rows ? c.more_wg_k : 1.0) * bzp * a_wg_k[a]) * 1e-3);
  const double a_bytes = (double)M * (double)K;
  if (a_bytes > k_stream_a_near) us = larger(us, 2.5 + a_bytes * (double)s.columns / (c.a_far * 1e7));
  return us + c.far * larger(a_bytes * 1e-6 - 4.0, 0.0) + c.b_far * larger((double)K * N * 1e-6 - c.b_near, 0.0);
}

// the row of k_stream_price for the kernel of 16 << i rows
const stream_price& stream_row(int i, const stream_shape& s, int M, int K) {
  if (s.sb <= 128) return k_stream_price[2 * i];
  if (s.far) return k_stream_price[10];
  if (i == 0 && K <= 16 * 64) return k_stream_price[7];
  if (i == 0 && M <= 4 && K > 64 * 64) return k_stream_price[6];
  if (i == 0 && K <= 32 * 64) return k_stream_price[9];
  if (i == 1 && K <= 32 * 64) return k_stream_price[8];
  return k_stream_price[2 * i + 1];
}

int price_select(int M, int N, int K, const call_form& f, double* price = nullptr) {
  int best = QG_KERNEL_TILE64;
  double best_us = 1e300;
  const auto take = [&](int kernel, double us) {
    if (us < best_us) best_us = us, best = kernel;
  };
  for (int i = 0; i < 3; ++i) {
    const stream_shape s = shape_of(16 << i, M, N, K);
    const stream_price& c = stream_row(i, s, M, K);
    if (s.row_blocks <= 65535) take(c.kernel, stream_price_us(c, s, M, N, K, f));
  }
  const bool few = qg_tile128_few(M, N, K);
  for (const tile_price& c : k_tile_price) {
    if (c.kernel == QG_KERNEL_TILE128 && (c.bn == 64) != few) continue;
    if (c.kernel == QG_KERNEL_TILE256 && K < 256) continue;  // 128 x 256 tiles there, without the loop priced here
    take(c.kernel, tile_price_us(c, M, N, K, f));
  }
  if (price != nullptr) *price = best_us;
  return best;
}

// fp32 activations in one launch, the streaming kernels quantizing what they stage (every column block converts its rows of A again):
//   conv, wg_c  per 16 rows: of a k block of a wave; of a workgroup, ns per 1 of K, where the chip is full
// against the 8-bit call plus a pass over A.  Fitted to 5000 drawn calls with M up to 512 and every form on each, the two launches as
// priced above; over 1200 others the choice is 1.0045 of the best form in the geometric mean, 41 of them slower by more than 5 %, 1.22 at
// worst.  Rows as of k_stream_price: in pairs, then 16 rows and up to 16 k blocks, 32 rows and up to 32.
struct f32_price {
  int kernel, rows;
  double fix, fix8, fix16, lat, crowd, block, conv, batch, second, wg, wg_k, wg_c, bzp_fix, k_fix, u8_fix, round, fetch, near;
};
const f32_price k_f32_price[] = {
    {QG_KERNEL_SKINNY16, 16, 3.073, 0.7941, 1.994, 0.0215, 0, 0.001986, 0.3066, 1.283, 0, 0, 0, 0, 0.001766, 0.05171,
     0.149, 0, 0.08193, 8.374},
    {QG_KERNEL_SKINNY16, 16, 0.1651, 3.949, 0.3, 0.000151, 3.551e-05, 0, 0.1556, 1.262, 0.002061, 2.118, 0.002785,
     0.004633, 0.07578, 0.117, 0.001036, 2.871, 0.1647, 7.094},
    {QG_KERNEL_SKINNY32, 32, 3.292, 0.1257, 0.2957, 0.7867, 6.27e-05, 0.0001959, 0.2005, 0.6206, 0, 0, 0, 0, 0.000607,
     0.1884, 0.07534, 0, 0.08566, 1.905},
    {QG_KERNEL_SKINNY32, 32, 4.393, 0.2841, 0.3, 0.1312, 0.4362, 0.002248, 0.2928, 0.5154, 0.02406, 5.859, 0.006754,
     0.001693, 0.02888, 0.04974, 0.1788, 0.003774, 0.04396, 3.747},
    {QG_KERNEL_SKINNY64, 64, 3.411, 0.1551, 0.3, 0.599, 0.00013, 6.944e-05, 0.2565, 0.8151, 0, 0, 0, 0, 4.335e-05,
     0.1963, 0.0003498, 0, 0.113, 0.7546},
    {QG_KERNEL_SKINNY64, 64, 3.138, 0.1427, 0.3, 0.483, 0.01722, 0.4916, 0.3054, 0.009889, 0.05034, 8.62, 0.008627,
     0.002157, 0.08039, 0.03217, 0, 2.353, 0.05803, 3.17},
    {QG_KERNEL_SKINNY16, 16, 1.438, 1.706, 0.3, 0.5419, 0.2651, 0, 0.1907, 0.6133, 0.1328, 1.962, 0, 0.006917,
     0.004586, 0.0676, 0.04746, 0.07502, 0.2399, 5.655},
    {QG_KERNEL_SKINNY32, 32, 2.977, 0.2696, 0.3, 0.02247, 0.06102, 0.3001, 0.2331, 0.004797, 0.07649, 6.056, 0.007601,
     0.001901, 0.01136, 0.1155, 0, 1.42, 0.141, 4.751},
};
const double k_quantize_fix = 1.666, k_quantize_mb = 1.165, k_quantize_most = 0.27;  // us; per million entries of A; up to so many

double f32_price_us(const f32_price& c, const stream_shape& s, int M, int N, int K, out_kind out, bool bzp) {
  const double g = ceil_div(M < c.rows ? M : c.rows, 4) / 4.0;
  const int near = s.columns < 8 ? s.columns : 8;
  double us = c.fix + (s.f.waves == 8 ? c.fix8 : s.f.waves == 16 ? c.fix16 : 0.0) + (bzp ? c.bzp_fix : 0.0) + (K % 64 != 0 ? c.k_fix : 0.0) +
              (out < OUT_F32 ? c.u8_fix : 0.0) + K / 1024.0 * (c.lat + c.crowd * share_of_chip(s.wgs)) + s.per * (c.block + c.conv * g) +
              s.batches * c.batch + c.fetch * larger(fetched_mb(s, M, N, K) + 3e-6 * near * M * K - c.near, 0.0);
  if (s.wgs > 256)
    us = larger(us * (1.0 + c.second) + (rounds_of(s.wgs) - 1.0) * c.round, 2.5 + (double)s.wgs * (c.wg + K * (c.wg_k + c.wg_c * g)) * 1e-3);
  return us;
}

// the row of k_f32_price for the kernel of 16 << i rows
const f32_price& f32_row(int i, const stream_shape& s, int K) {
  if (s.sb <= 128) return k_f32_price[2 * i];
  return k_f32_price[i == 0 && K <= 16 * 64 ? 6 : i == 1 && K <= 32 * 64 ? 7 : 2 * i + 1];
}

const int k_f32_most_rows = 512;  // 64 rows at a time, A would be converted by every column block for each of many row blocks

// the best kernel for one launch; best_us: what it has to beat, or QG_KERNEL_AUTO is the answer
int f32_one_launch(int M, int N, int K, const call_form& f, double best_us) {
  int best = QG_KERNEL_AUTO;
  for (int i = 0; i < 3; ++i) {
    const stream_shape s = shape_of(16 << i, M, N, K);
    const f32_price& c = f32_row(i, s, K);
    const double us = f32_price_us(c, s, M, N, K, f.out, f.bzp);
    if (us < best_us) best_us = us, best = c.kernel;
  }
  return best;
}

// the kernel for one launch, or QG_KERNEL_AUTO where two launches are estimated to be faster
int f32_select(int M, int N, int K, const call_form& f) {
  if (M > k_f32_most_rows) return QG_KERNEL_AUTO;
  double best_us;
  price_select(M, N, K, f, &best_us);
  const double entries = (double)M * (double)K * 1e-6;
  return f32_one_launch(M, N, K, f, best_us + k_quantize_fix + k_quantize_mb * (entries < k_quantize_most ? entries : k_quantize_most));
}

// Outlier-split weights in a call without a workspace: terms as of k_stream_price, and
//   sp, more            per batch and column of a wave: any outliers; for every 64 of them beyond the first
//   wg_sp, wg_more      the same where the chip is full, ns per workgroup and 1 of K; wg_more per 1 % of outliers
// Per kernel a row for up to 128 super-blocks of rows x 32 columns, up to 256 and more.  Fitted to 5000 drawn calls (M 1 .. 512, N and K
// 64 .. 12288, up to 10 % of outliers); over 1200 others the choice is 1.002 of the best kernel in the geometric mean, 22 by more than
// 5 %, 1.18 at worst.  The former constants, below, 1.015, 592 of 6200 and 1.73: they are of kernels with another sparse term.
struct split_price {
  int kernel, rows;
  double fix, fix8, fix16, lat, crowd, block, batch, sp, more, second, wg, wg_k, wg_sp, wg_more, round;
  double bzp_fix, fix4, fix1, f32_fix, f32_wg, i32_fix, i32_wg;
};
const split_price k_split_price[] = {
    {QG_KERNEL_SKINNY16, 16, 2.485, 0.007827, 0.4168, 0.2054, 0.1653, 0.003457, 0.2409, 0.2594, 0.09838, 0, 0, 0, 0, 0,
     0, 0.002537, 0.0109, 0.1063, 0.04752, 0, 2.446e-05, 0},
    {QG_KERNEL_SKINNY16, 16, 1.752, 0.6388, 0.9435, 0.166, 0.4928, 0.003034, 0.369, 0.393, 0.1301, 0.06173, 0.907,
     0.0002001, 0.0004947, 9.921e-05, 0.2166, 3.449e-05, 7.298e-05, 0.02186, 0.005837, 0.1272, 2.765e-05, 0.0676},
    {QG_KERNEL_SKINNY16, 16, 1.89, 0.1, 0.3, 0.3568, 0.2379, 0.0008896, 0.6251, 0.1649, 0.08464, 0.2748, 0.6685,
     0.001008, 0.0002278, 0.0001061, 0.2239, 0.06024, 0.1226, 0.1455, 0.001569, 0.01837, 0, 0.0001049},
    {QG_KERNEL_SKINNY32, 32, 2.77, 0.08423, 0.2733, 0.3434, 0.169, 0.006214, 0.1397, 0.2137, 0.1076, 0, 0, 0, 0, 0, 0,
     0.07214, 0.05136, 0.3462, 0.01976, 0, 5.08e-05, 0},
    {QG_KERNEL_SKINNY32, 32, 3.142, 0.09819, 0.3, 0.1572, 0.67, 0.001538, 0.5676, 0.2399, 0.1337, 0.3, 4, 0.002,
     0.0005, 0.0002, 0.5, 0.0005637, 0, 0.01894, 0.005244, 0.001, 6.265e-05, 0.001},
    {QG_KERNEL_SKINNY32, 32, 1.214, 0.1, 0.3, 0.6091, 0.4061, 0.0187, 0.3597, 0.1358, 0.1242, 0.1712, 0.4243, 0.002043,
     0.000657, 0.0001401, 0.6441, 2.85e-05, 2.289e-05, 0.4325, 0.06362, 0.01155, 0.03444, 0.2135},
    {QG_KERNEL_SKINNY64, 64, 2.868, 0.07966, 0.3, 0.256, 0.5971, 0.01902, 0.3058, 0.2105, 0.2004, 0, 0, 0, 0, 0, 0,
     0.0005317, 0.1179, 0.1774, 0.07447, 0, 0.1116, 0},
    {QG_KERNEL_SKINNY64, 64, 3.211, 0.08918, 0.3, 0.8051, 0.2196, 0.01089, 0.09034, 0.2015, 0.1958, 0.3, 4, 0.002,
     0.0005, 0.0002, 0.5, 0, 0.02823, 0.1422, 0.2584, 0.001, 1.034, 0.001},
    {QG_KERNEL_SKINNY64, 64, 2.806, 0.8921, 0.3, 0.2751, 0.1834, 0.06699, 0.6894, 0.2093, 0.6949, 0.4064, 8.089,
     0.00487, 0.001473, 0.0004593, 0.2568, 0.7752, 0.000188, 1.409, 1.694, 3.591, 0.0001071, 1.391},
};

// outliers: their share of the weights
double split_price_us(const split_price& c, const stream_shape& s, int K, double outliers, const call_form& f) {
  const double any = outliers > 0.0 ? 1.0 : 0.0;
  const double out_fix[] = {0.0, 0.0, c.f32_fix, c.i32_fix}, out_wg[] = {0.0, 0.0, c.f32_wg, c.i32_wg};
  const double fix = c.fix + (s.f.waves == 8 ? c.fix8 : s.f.waves == 16 ? c.fix16 : 0.0) + out_fix[f.out] + (f.bzp ? c.bzp_fix : 0.0) +
                     (f.a_align == 16 ? 0.0 : f.a_align == 4 ? c.fix4 : c.fix1);
  const double us = fix + K / 1024.0 * (c.lat + c.crowd * share_of_chip(s.wgs)) + s.per * c.block + s.batches * c.batch +
                    (s.batches + 1) * s.f.columns * (any * c.sp + larger(outliers * 1024.0 * s.f.batch - 64.0, 0.0) / 64.0 * c.more);
  if (s.wgs <= 256) return us;
  return larger(us * (1.0 + c.second) + (rounds_of(s.wgs) - 1.0) * c.round,
                2.5 + (double)s.wgs * (c.wg + out_wg[f.out] + K * (c.wg_k + any * c.wg_sp + outliers * 100.0 * c.wg_more)) * 1e-3);
}

int split_select(int M, int N, int K, double outliers, const call_form& f) {
  int best = QG_KERNEL_SKINNY64;
  double best_us = 1e300;
  for (int i = 0; i < 3; ++i) {
    const stream_shape s = shape_of(16 << i, M, N, K, true);
    const split_price& c = k_split_price[3 * i + (s.sb > 256 ? 2 : s.sb > 128 ? 1 : 0)];
    const double us = split_price_us(c, s, K, outliers, f);
    if (s.row_blocks <= 65535 && us < best_us) best_us = us, best = c.kernel;
  }
  return best;
}

// What the queries about K splits and workspaces of outlier-split weights go by, and calls that ask for a split or bring a workspace for one
// (one answer for a shape; the constants are of the time when these weights always ran on sixteen waves)
const stream_cost k_stream_cost_16wave[] = {
    {QG_KERNEL_SKINNY16, 16, 3.58, 7.3e-5, 7.55, 0.74e-3},
    {QG_KERNEL_SKINNY32, 32, 4.13, 1.99e-4, 10.33, 1.28e-3},
    {QG_KERNEL_SKINNY64, 64, 4.96, 3.88e-4, 14.26, 2.23e-3},
};
// The dense convolution: the tile loops with the im2col addressing folded into the requests, the streaming kernels with
// per-lane tap addressing (Cin % 16 == 0), and for "same" layers (stride 1, output as large as the input, Cin % 32 == 0) the kernels
// that keep the input patch of a pixel tile in LDS.  Formulas as for the GEMM, with
//   chunk       channel counts off 64, whose requests keep a tap per lane;  tap: 64 / Cin of the steps begin a new tap
//   load        per KiB of patch;  half: channel counts off 64, whose last slab is half full
//   pass        what does not run side by side, the LDS of a wide patch allowing few workgroups per CU, runs one after the
//               other, each pass at so much of the pace of a workgroup alone
// Fitted to 20690 layers (1 x 1 to 7 x 7, stride 1 and 2, 16 .. 512 channels in, 8 .. 512 out, 5 .. 200 pixels wide, 1 .. 32 images) as
// the GEMM's; the streaming kernels' terms again to 5000 layers when these kernels got faster and took channel counts off 64.  Over
// 1500 others the choice is 1.005 of the best kernel in the mean, 1.37 at worst, 48 by more than 5 % (the former terms: 1.028).
struct conv_tile_price {
  int kernel, bm, bn;
  double fix, lat, crowd, thr, fill, epi, out, rag_fix, rag_epi, chunk_fix, chunk_lat, chunk_thr, bzp_fix, tap_lat, tap_thr, tall, bzp_lat, bzp_thr;
};
struct conv_stream_price {
  int kernel, rows;
  double fix, fix8, fix16, lat, crowd, block, batch, second, wg, wg_k, bzp_fix, bzp_lat, rag_fix, rag_wg;
  double chunk_fix, chunk_lat, chunk_wg_k, a_far, round, far, fetch, near;
};
struct conv_patch_price {
  int kernel, bm, bn;
  double fix, lat, crowd, thr, fill, epi, rag_fix, rag_epi, load, load_thr, bzp_fix, bzp_load, half_lat, half_thr, pass;
};
const conv_tile_price k_conv_tile_price[] = {
    {QG_KERNEL_TILE64K1, 64, 64, 2.621, 0.2996, 0.02843, 0.1181, 0, 0.3721, 1.687, 0.2414, 0.2388, 0.4666, 1.296, 1.17,
     0.1126, 0.003831, 0, 0.1076, 0.09862, 0.1185},
    {QG_KERNEL_TILE64, 64, 64, 3.379, 0.1517, 0.01472, 0.09318, 0.1842, 1.269, 3, 0.2444, 0.1268, 0.66, 1.219, 1.347,
     0.01917, 0.09827, 0.1015, 0.1107, 0.05257, 0.09864},
    {QG_KERNEL_TILE64K4, 64, 64, 4.535, 0.0883, 0.01584, 0.1078, 0.08981, 2.688, 3, 0.2518, 0.2099, 0.952, 1.272, 1.526,
     0.08897, 0.7561, 0.5257, 0.1444, 0.05258, 0.0748},
    {QG_KERNEL_TILE64X32K8, 64, 32, 5, 0.06172, 0.01282, 0.07016, 0.5492, 3.366, 3, 0.2932, 0.5349, 0.6883, 2.437, 2.334,
     0.2064, 0.8822, 0.7738, 0.1045, 0.03078, 0.09294},
    {QG_KERNEL_TILE128, 128, 128, 4.395, 0.1804, 0.05482, 0.2991, 0.6572, 1.667, 3, 0.4675, 1.152, 0.1934, 3.203, 1.21,
     0.07541, 0.7189, 0.1407, 0.2448, 0.08744, 0.08856},
    {QG_KERNEL_TILE128X256, 128, 256, 6.375, 0.1898, 0.1673, 0.4174, 0.5815, 3.169, 3, 1.243, 1.684, 0.1547, 3.392,
     1.611, 0.02083, 1.924, 0.4226, 0.148, 0.05569, 0.0766},
};
// (in pairs, as for the GEMM: up to 128 super-blocks, where the terms for more workgroups than CUs are left out, and more)
const conv_stream_price k_conv_stream_price[] = {
    {QG_KERNEL_SKINNY16, 16, 3.179, 0.3758, 1.25, 0.0008043, 0.129, 0.193, 0.2321, 0, 0, 0, 0.0001065, 0, 0.004859, 0, 1.219,
     0.002297, 0, 1, 0, 0.000076, 0.008103, 33.75},
    {QG_KERNEL_SKINNY16, 16, 2.683, 1.776, 0.5, 0.0007659, 0.0003954, 0.001798, 0.7578, 0.186, 0.05215, 0.003142, 0.0004539,
     0.0004355, 0.08225, 0.2894, 0.6832, 1.101, 0.9658, 1, 0.7804, 0.01493, 0.08158, 7.564},
    {QG_KERNEL_SKINNY32, 32, 3.643, 0.1328, 1.176, 0.006866, 0.2389, 0.3819, 0.3824, 0, 0, 0, 0.01993, 0.000073, 0.08501, 0,
     1.243, 0.4892, 0, 1, 0, 0.000071, 0.0008134, 86.16},
    {QG_KERNEL_SKINNY32, 32, 4.389, 0.4313, 0.5, 0.009968, 0.02833, 0.1809, 0.3108, 0.0001235, 14.3, 0.00007, 0.0001865,
     0.0001123, 0.2391, 0.1688, 0.6232, 1.411, 26.8, 0.8277, 2.836, 0.0106, 0.02866, 40.14},
    {QG_KERNEL_SKINNY64, 64, 4.178, 0.1899, 0.5, 1.299, 0.4995, 0.01924, 0.00214, 0, 0, 0, 0.0149, 0.02231, 0.2289, 0, 0.5228,
     1.317, 0, 1.009, 0, 0.000079, 0.01025, 0.01546},
    {QG_KERNEL_SKINNY64, 64, 5.054, 0.2298, 0.5, 0.002852, 0.01836, 0.5464, 0.1645, 0.5519, 15.89, 0.006494, 0.02185, 0.00237,
     0.1778, 0.003916, 0.09427, 1.519, 1.309, 0.6592, 0.2777, 0.007927, 0.03492, 0.2291},
};
const conv_patch_price k_conv_patch_price[] = {
    {QG_KERNEL_PATCH64X128, 64, 128, 3.4, 0.0935, 0.03727, 0.1396, 0.8133, 1.005, 2.676, 3.501, 0.05252, 0.01825, 0.9731,
     0.01964, 2.868, 0.8962, 0.9737},
    {QG_KERNEL_PATCH128X64, 128, 64, 3.641, 0.1496, 0, 0.0842, 0.3523, 0.8482, 2.736, 2.735, 0.005236, 0.02926, 0.8379,
     0.008291, 1.219, 1.102, 1.135},
    {QG_KERNEL_PATCH256X64, 256, 64, 4.05, 0.1615, 0.001215, 0.1679, 0.2977, 1.637, 6.579, 5.846, 0.01247, 0.009308,
     0.5507, 0.0143, 1.23, 1.17, 1.195},
    {QG_KERNEL_PATCH256, 256, 128, 6.063, 0.2323, 0.0866, 0.2649, 0.2914, 3.118, 13.86, 13.33, 0.001793, 0, 1.036,
     0.01437, 1.206, 1.216, 1.103},
    {QG_KERNEL_PATCH512, 512, 128, 9.67, 0.3225, 0.2546, 0.5183, 0.2761, 7.22, 17.92, 33.57, 0.003051, 0.0001414, 1.853,
     0.01148, 1.254, 0.574, 1.019},
};
// ... and the builds of QG_KERNEL_PATCH64X128 for at most one tile per CU, with four and two wave sets
const conv_patch_price k_conv_few4_price =
    {QG_KERNEL_PATCH64X128, 64, 64, 4.671, 0.05276, 0.01044, 0, 0, 0, 1.732, 0, 0.0001684, 0, 0.8553, 0.01451, 1.15, 0,
     0};
const conv_patch_price k_conv_few2_price =
    {QG_KERNEL_PATCH64X128, 64, 128, 4.087, 0.08389, 0.01578, 0, 0, 0, 4.864, 0, 0.01644, 0, 0.9648, 0.009549, 1.266, 0,
     0};

double conv_tile_us(const conv_tile_price& c, const qg_gemm_args& a) {
  const double kt = (double)ceil_div(a.K, 64), wgs = (double)ceil_div(a.M, c.bm) * (double)ceil_div(a.N, c.bn), M = a.M, N = a.N;
  const bool chunk = a.cv_Cin % 64 != 0, rag = a.c_vec == 0;
  const double tap = 64.0 / a.cv_Cin;
  const double fix = c.fix + (rag ? c.rag_fix : 0.0) + (a.has_bzp ? c.bzp_fix : 0.0) + (chunk ? c.chunk_fix : 0.0);
  const double lat = c.lat * (chunk ? c.chunk_lat : 1.0 + c.tap_lat * tap) * (a.has_bzp ? 1.0 + c.bzp_lat : 1.0) * (1.0 + c.tall * M / (M + N));
  const double alone = fmax(fix + kt * (lat + c.crowd * fmin(wgs, 256.0) / 256.0), 2.5 + M * N / (c.out * 1e6));
  if (wgs <= 256.0) return alone;
  const double rounds = ceil(wgs / 256.0), steps = rounds + c.fill * (wgs / 256.0 - rounds);
  const double thr = c.thr * (chunk ? c.chunk_thr : 1.0 + c.tap_thr * tap) * (a.has_bzp ? 1.0 + c.bzp_thr : 1.0);
  return fmax(alone, 2.5 + rounds * (c.epi + (rag ? c.rag_epi : 0.0)) + steps * kt * thr);
}

double conv_stream_us(const conv_stream_price& c, const qg_gemm_args& a) {
  const stream_shape s = shape_of(c.rows, a.M, a.N, a.K);
  const bool chunk = a.cv_Cin % 64 != 0, rag = a.c_vec == 0;
  const double bzp = a.has_bzp ? 1.0 + c.bzp_lat : 1.0;
  double us = c.fix + (s.f.waves == 8 ? c.fix8 : s.f.waves == 16 ? c.fix16 : 0.0) + (rag ? c.rag_fix : 0.0) + (a.has_bzp ? c.bzp_fix : 0.0) +
              (chunk ? c.chunk_fix : 0.0) +
              (a.K / 1024.0 * (c.lat + c.crowd * share_of_chip(s.wgs)) + s.per * c.block + s.batches * c.batch) * bzp * (chunk ? c.chunk_lat : 1.0) +
              c.fetch * fmax(fetched_mb(s, a.M, a.N, a.K) - c.near, 0.0);
  if (s.wgs > 256)
    us = fmax(us * (1.0 + c.second) + (rounds_of(s.wgs) - 1.0) * c.round,
              2.5 + (double)s.wgs * (c.wg + (rag ? c.rag_wg : 0.0) + a.K * c.wg_k * bzp * (chunk ? c.chunk_wg_k : 1.0)) * 1e-3);
  const double a_bytes = (double)a.M * (double)a.K;
  if (a_bytes > k_stream_a_near) us = fmax(us, 2.5 + a_bytes * (double)s.columns / (c.a_far * 1e7));
  return us + c.far * fmax(a_bytes * 1e-6 - 4.0, 0.0);
}

double conv_patch_us(const conv_patch_price& c, const qg_gemm_args& a, int per_cu) {
  const double kt = (double)ceil_div(a.K, 64), wgs = (double)ceil_div(a.M, c.bm) * (double)ceil_div(a.N, c.bn);
  const bool half = a.cv_Cin % 64 != 0;
  const double kb = ((double)c.bm + (double)(a.cv_R - 1) * a.cv_W + a.cv_R - 1) * a.cv_Cin / 1024.0;
  const double rag = a.c_vec ? 0.0 : fmin((double)a.N / c.bn, 1.0), bzp = a.has_bzp ? 1.0 : 0.0;
  const double alone = c.fix + rag * c.rag_fix + bzp * (c.bzp_fix + kb * c.bzp_load) + kb * c.load +
                       kt * (c.lat * (half ? c.half_lat : 1.0) + c.crowd * fmin(wgs, 256.0) / 256.0);
  if (wgs <= 256.0) return alone;
  const double rounds = ceil(wgs / 256.0), steps = rounds + c.fill * (wgs / 256.0 - rounds), passes = ceil(wgs / (256.0 * per_cu));
  const double full = 2.5 + rounds * (c.epi + rag * c.rag_epi + kb * c.load_thr + bzp * kb * c.bzp_load) +
                      steps * kt * c.thr * (half ? c.half_thr : 1.0);
  return fmax(fmax(alone, full), passes > 1.0 ? 2.5 + passes * (alone - 2.5) * c.pass : 0.0);
}

int select_stream_kernel(int M, int N, int K) {
  int best = QG_KERNEL_SKINNY64;
  double best_us = 1e300;
  for (const stream_cost& c : k_stream_cost_16wave) {
    const long long blocks = ceil_div(M, c.rows);
    if (blocks > 65535) continue;
    const double us = stream_estimate(c, M, N, K, false);
    if (us < best_us) best_us = us, best = c.kernel;
  }
  return best;
}

// the caller's rule for the shape, or QG_KERNEL_AUTO
int rule_kernel(int M, int N, int K) {
  for (int i = 0; i < g_nrules; ++i) {
    const qg_dispatch_rule& r = g_rules[i];
    if (M >= r.m_lo && M <= r.m_hi && N >= r.n_lo && N <= r.n_hi && K >= r.k_lo && K <= r.k_hi) return r.kernel;
  }
  return QG_KERNEL_AUTO;
}

hipError_t launch_rows(const qg_gemm_args& a, int mode, int kernel, hipStream_t s) {
  if (kernel <= QG_KERNEL_SKINNY64) return qg_launch_gemm_skinny(a, mode, kernel, s);
  return qg_launch_gemm_tile(a, mode, kernel, s);
}

// The kernels address A with 32-bit byte offsets from its base.  An A beyond that reach is run as several
// launches over consecutive row ranges (whole 256-row tiles where possible, so the tiling is that of one launch),
// each with its own base pointers; rows are independent, the result is the same.
hipError_t launch_gemm(const qg_gemm_args& a, int mode, int kernel, hipStream_t s) {
  const uint64_t reach = (1ull << 32) - (uint64_t)a.K - 4096;
  if ((uint64_t)(a.M - 1) * (uint64_t)a.lda < reach) return launch_rows(a, mode, kernel, s);
  int rows = (int)(reach / (uint64_t)a.lda);  // >= 1: lda is an int
  if (rows >= 256) rows = rows / 256 * 256;
  for (int r0 = 0; r0 < a.M; r0 += rows) {
    qg_gemm_args b = a;
    b.M = a.M - r0 < rows ? a.M - r0 : rows;
    b.A = a.A + (size_t)r0 * (size_t)a.lda;
    if (a.C) b.C = a.C + (size_t)r0 * (size_t)a.ldc;
    if (a.Cf) b.Cf = a.Cf + (size_t)r0 * (size_t)a.ldc;
    if (a.C32) b.C32 = a.C32 + (size_t)r0 * (size_t)a.ldc;
    if (a.rowsum_out) b.rowsum_out = a.rowsum_out + r0;
    const hipError_t e = launch_rows(b, mode, kernel, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// kernel id valid for this M (the streaming kernels put row blocks on the 16-bit grid dimension)
bool kernel_ok(int kernel, int M) {
  if (kernel < QG_KERNEL_AUTO || kernel > QG_KERNEL_LAST) return false;
  if (kernel >= QG_KERNEL_SKINNY16 && kernel <= QG_KERNEL_SKINNY64)
    return ceil_div(M, 16 << (kernel - QG_KERNEL_SKINNY16)) <= 65535;
  return true;
}

// resolves QG_KERNEL_AUTO for a descriptor and checks an explicit choice against it: QG_OK, or
// QG_EINVAL (unknown id / too many row blocks), QG_EUNSUPPORTED (tiled kernel on a split descriptor)
int resolve_kernel(const qg_packed_b* Bp, int M, int* kernel) {
  if (!kernel_ok(*kernel, M)) return QG_EINVAL;
  if (Bp->split) {
    if (*kernel == QG_KERNEL_AUTO) *kernel = select_stream_kernel(M, Bp->N, Bp->K);
    if (*kernel > QG_KERNEL_SKINNY64) return QG_EUNSUPPORTED;
    return kernel_ok(*kernel, M) ? QG_OK : QG_EINVAL;
  }
  if (*kernel == QG_KERNEL_AUTO) *kernel = rule_kernel(M, Bp->N, Bp->K);
  if (*kernel == QG_KERNEL_AUTO || !kernel_ok(*kernel, M)) *kernel = builtin_select(M, Bp->N, Bp->K);
  return QG_OK;
}

// ---- K split across workgroups (streaming kernels; the caller's workspace is the paper's C_buffer, Appendix A)
constexpr int kSlotInts = 64 * 4 + 16;   // one (K slice, row block of 16) slot: 64 lanes x 4 partial sums + 16 row sums
constexpr int kMaxKsplit = 64;

struct splitk_layout {
  size_t cnt_ints, slot_ints;
  size_t bytes() const { return (cnt_ints + slot_ints) * sizeof(int32_t); }
};
// counters first (one per row block of 16 and fragment column, rounded up to 256 bytes), then the slots
splitk_layout splitk_ws(int kernel, int M, int N, int ksplit) {
  if (kernel == QG_KERNEL_TILE128) {  // one counter per 128 x 128 tile; a slot is 256 threads x (64 sums + 2 row offsets)
    const size_t tiles = (size_t)ceil_div(M, 128) * (size_t)ceil_div(N, 128);
    return {(tiles + 63) / 64 * 64, tiles * (size_t)ksplit * (66 * 256)};
  }
  const int rows = 16 << (kernel - QG_KERNEL_SKINNY16);
  const size_t units = (size_t)ceil_div(M, rows) * (size_t)(2 * ceil_div(N, 32)) * (size_t)(rows / 16);
  return {(units + 63) / 64 * 64, units * (size_t)ksplit * kSlotInts};
}
// slices that are all non-empty: at most one per 64-deep block of K (a pair of blocks for 4-bit weights)
int clamp_ksplit(const qg_packed_b* Bp, int ksplit) {
  const int blocks = Bp->K_pad / QG_FRAG_K / (Bp->split ? 2 : 1);
  if (ksplit > blocks) ksplit = blocks;
  const int per = ceil_div(blocks, ksplit);
  return ceil_div(blocks, per);
}
// Built-in choice of the split, from timings of 16 x {16..512} x {4096..32768} and 64 x {64, 256} x {8192, 16384}
// (cold weights): handing a partial tile through the workspace costs 1.5 - 2 us, so a split pays only where it
// removes several batches of weight loads from every wave's chain.  Give each wave of a slice four 64-deep blocks
// (one batch of loads); take the split from 4 slices up (from 2 for 64-row blocks, whose waves do four times the
// work per block), and never more slices than there are idle CUs to take them.
// The 128 x 128 tile: slices of whole 64-deep tiles, at least four each (the depth of the hand-scheduled loop's
// pipeline), K a multiple of 64, dense weights.  -> the number of slices that `ksplit` gives, 1 if it cannot be split
int clamp_ksplit_tile128(const qg_packed_b* Bp, int ksplit) {
  if (Bp->split || Bp->K % QG_FRAG_K != 0) return 1;
  const int blocks = Bp->K / QG_FRAG_K;
  if (ksplit > blocks / 4) ksplit = blocks / 4;
  while (ksplit > 1) {
    const int per = ceil_div(blocks, ksplit), s = ceil_div(blocks, per);
    if (blocks - (s - 1) * per >= 4) return s;
    --ksplit;
  }
  return 1;
}
int auto_ksplit(int kernel, int M, const qg_packed_b* Bp) {
  if (kernel < QG_KERNEL_SKINNY16 || kernel > QG_KERNEL_SKINNY64) return 1;
  const int rows = 16 << (kernel - QG_KERNEL_SKINNY16);
  const long long wgs = (long long)ceil_div(M, rows) * (2 * ceil_div(Bp->N, 32));
  if (wgs * 2 > 256) return 1;
  int s = Bp->K_pad / QG_FRAG_K / (16 * 4);  // 16 waves x 4 blocks (slices on fewer waves have as many more each)
  if (s > 256 / wgs) s = (int)(256 / wgs);
  if (s > 16) s = 16;
  if (s < (rows == 64 ? 2 : 4)) return 1;
  return clamp_ksplit(Bp, s);
}
// QG_KERNEL_AUTO of one call.  A call that leaves kernel and split to the library and brings no workspace, or one that no
// query asked for, gets the kernel of the closer prices, without a split (a split that the queries did not announce
// must not be used: the caller's workspace may be anything).  All others get what the queries answer for.
int resolve_call(const qg_packed_b* Bp, int M, int* kernel, int* ksplit, const call_form& f, const void* workspace_dev) {
  if (*kernel != QG_KERNEL_AUTO || *ksplit < 0 || *ksplit > 1 || M <= 0) return resolve_kernel(Bp, M, kernel);
  if (Bp->split) {
    if (*ksplit == 0 && workspace_dev != nullptr) {
      const int k = select_stream_kernel(M, Bp->N, Bp->K);
      if (auto_ksplit(k, M, Bp) > 1) return resolve_kernel(Bp, M, kernel);
      *ksplit = 1;
    }
    const int k = split_select(M, Bp->N, Bp->K, (double)Bp->nnz / ((double)Bp->N * Bp->K), f);
    if (!kernel_ok(k, M)) return resolve_kernel(Bp, M, kernel);  // (too many row blocks for any)
    return *kernel = k, QG_OK;
  }
  const int rule = rule_kernel(M, Bp->N, Bp->K);
  if (rule != QG_KERNEL_AUTO && kernel_ok(rule, M)) return *kernel = rule, QG_OK;
  if (*ksplit == 0 && workspace_dev != nullptr) {
    const int k = builtin_select(M, Bp->N, Bp->K);
    if (auto_ksplit(k, M, Bp) > 1) return *kernel = k, QG_OK;
    *ksplit = 1;
  }
  *kernel = price_select(M, Bp->N, Bp->K, f);
  return QG_OK;
}
int a_align(const uint8_t* A_dev, int lda) {
  return aligned(A_dev, 16) && lda % 16 == 0 ? 16 : aligned(A_dev, 4) && lda % 4 == 0 ? 4 : 1;
}
out_kind u8_kind(const uint8_t* C_dev, int ldc) { return aligned(C_dev, 16) && ldc % 16 == 0 ? OUT_U8 : OUT_U8_RAGGED; }
// ksplit_req: 0 = built-in choice (1 without a workspace), otherwise the caller's.  Fills the workspace fields of `a`.
int resolve_ksplit(const qg_packed_b* Bp, int M, int kernel, int ksplit_req, void* workspace_dev, size_t workspace_bytes,
                   bool bytes_known, qg_gemm_args* a) {
  a->ksplit = 1;
  a->ks_per = Bp->K_pad / QG_FRAG_K;
  a->ws_cnt = a->ws_slots = nullptr;
  if (ksplit_req < 0 || ksplit_req > kMaxKsplit) return QG_EINVAL;
  if (M == 0) return QG_OK;
  int s = ksplit_req;
  if (kernel == QG_KERNEL_TILE128 && s > 1) {
    // the caller's split on the 128 x 128 tile (never the built-in choice)
    s = clamp_ksplit_tile128(Bp, s);
    if (s <= 1) return QG_OK;
    if (!workspace_dev) return QG_EWORKSPACE;
    if (!aligned(workspace_dev, 16)) return QG_EALIGN;
    const splitk_layout w = splitk_ws(kernel, M, Bp->N, s);
    if (bytes_known && workspace_bytes < w.bytes()) return QG_EWORKSPACE;
    a->ksplit = s;
    a->ks_per = ceil_div(Bp->K / QG_FRAG_K, s);
    a->ws_cnt = static_cast<int32_t*>(workspace_dev);
    a->ws_slots = a->ws_cnt + w.cnt_ints;
    return QG_OK;
  }
  if (kernel > QG_KERNEL_SKINNY64) {
    if (s > 1) return QG_EUNSUPPORTED;  // the other tiled kernels keep K inside the workgroup
    return QG_OK;
  }
  if (s == 0) s = workspace_dev ? auto_ksplit(kernel, M, Bp) : 1;
  s = clamp_ksplit(Bp, s);
  if (s <= 1) return QG_OK;
  if (!workspace_dev) return QG_EWORKSPACE;
  if (!aligned(workspace_dev, 16)) return QG_EALIGN;
  const splitk_layout w = splitk_ws(kernel, M, Bp->N, s);
  if (bytes_known && workspace_bytes < w.bytes()) return QG_EWORKSPACE;
  a->ksplit = s;
  {
    const int unit = Bp->split ? 2 : 1, blocks = Bp->K_pad / QG_FRAG_K / unit;
    a->ks_per = ceil_div(blocks, s) * unit;
  }
  a->ws_cnt = static_cast<int32_t*>(workspace_dev);
  a->ws_slots = a->ws_cnt + w.cnt_ints;
  return QG_OK;
}

// ---- built-in scratch for callers that cannot allocate (qg_gemm_u8s8_requant_noalloc) -------------------------
// The K-split workspace as a file-scope device array: every GPU the library runs on holds its own copy, at its own
// address, from the moment the code object is loaded until the process ends.  Zero-initialised at load, and every
// call leaves the ticket counters at zero, so no clearing pass is needed between calls.  In host code the array's
// name is only a handle: the device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) int32_t qg_noalloc_scratch[QG_NOALLOC_SCRATCH_BYTES / sizeof(int32_t)];
void* g_scratch_ptr[64] = {nullptr};  // per device; concurrent first calls may both look it up (same answer)

int noalloc_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return QG_ELAUNCH;
  if (dev < 0 || dev >= 64) return QG_EUNSUPPORTED;
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(qg_noalloc_scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return QG_ELAUNCH;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return QG_OK;
}

__global__ void qg_fill_zero_kernel(int32_t* p, size_t n) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = 0;
}

}  // namespace

extern "C" {

const char* qg_kernel_name(int kernel) {
  static const char* const names[] = {"auto",   "skinny16", "skinny32",    "skinny64",
                                      "tile64", "tile128",  "tile128x256", "tile256",
                                      "tile64k4", "tile64k1", "tile64x32k8",
                                      "patch64x128", "patch128x64", "patch256x64", "patch256", "patch512"};
  return (kernel >= 0 && kernel <= QG_KERNEL_CONV_LAST) ? names[kernel] : nullptr;
}

int qg_kernel_select(int M, int N, int K) {
  if (M <= 0 || N <= 0 || K <= 0) return QG_EINVAL;
  const int rule = rule_kernel(M, N, K);
  if (rule != QG_KERNEL_AUTO && kernel_ok(rule, M)) return rule;
  return price_select(M, ceil_div(N, 16) * 16, ceil_div(K, 64) * 64, {16, OUT_U8, false});
}

int qg_dispatch_set_rules(const qg_dispatch_rule* rules_host, int n) {
  if (n < 0 || n > QG_MAX_DISPATCH_RULES) return QG_EINVAL;
  if (n > 0 && !rules_host) return QG_ENULL;
  for (int i = 0; i < n; ++i) {
    const qg_dispatch_rule& r = rules_host[i];
    if (r.m_lo > r.m_hi || r.n_lo > r.n_hi || r.k_lo > r.k_hi) return QG_EINVAL;
    if (r.kernel < QG_KERNEL_SKINNY16 || r.kernel > QG_KERNEL_LAST) return QG_EINVAL;
  }
  for (int i = 0; i < n; ++i) g_rules[i] = rules_host[i];
  g_nrules = n;
  return QG_OK;
}

const char* qg_status_string(int code) {
  switch (code) {
    case QG_OK: return "ok";
    case QG_ENULL: return "required pointer is NULL";
    case QG_EINVAL: return "invalid size, leading dimension, zero point or count";
    case QG_EALIGN: return "device pointer alignment violated";
    case QG_EWORKSPACE: return "workspace required but not provided";
    case QG_ELAUNCH: return "HIP runtime refused the launch or copy";
    case QG_ENOMEM: return "host allocation failed";
    case QG_EUNSUPPORTED: return "configuration not implemented in this build";
    case QG_ECAPACITY: return "more outliers than the sparse buffer holds";
    default: return "unknown status";
  }
}

int qg_pack_b_sizes(int K, int N, size_t* packed_bytes, size_t* col_offsets_bytes) {
  if (!packed_bytes || !col_offsets_bytes) return QG_ENULL;
  if (K <= 0 || N <= 0 || K > QG_MAX_K) return QG_EINVAL;
  const size_t K_pad = (size_t)qg_round_up(K, QG_KPAD), N_pad = (size_t)qg_round_up(N, QG_NPAD);
  *packed_bytes = K_pad * N_pad;
  *col_offsets_bytes = 2 * N_pad * sizeof(int32_t);
  return QG_OK;
}

static int pack_b_any(const int8_t* B_dev, int K, int N, int ldb, int transposed, const int32_t* b_zp_host,
                      int n_b_zp, void* packed_dev, int32_t* col_offsets_dev, void* stream, qg_packed_b** out);

int qg_pack_b(const int8_t* B_dev, int K, int N, int ldb, const int32_t* b_zp_host, int n_b_zp,
              void* packed_dev, int32_t* col_offsets_dev, void* stream, qg_packed_b** out) {
  return pack_b_any(B_dev, K, N, ldb, 0, b_zp_host, n_b_zp, packed_dev, col_offsets_dev, stream, out);
}

int qg_pack_b_transposed(const int8_t* Bt_dev, int K, int N, int ldbt, const int32_t* b_zp_host, int n_b_zp,
                         void* packed_dev, int32_t* col_offsets_dev, void* stream, qg_packed_b** out) {
  return pack_b_any(Bt_dev, K, N, ldbt, 1, b_zp_host, n_b_zp, packed_dev, col_offsets_dev, stream, out);
}

static int pack_b_any(const int8_t* B_dev, int K, int N, int ldb, int transposed, const int32_t* b_zp_host,
                      int n_b_zp, void* packed_dev, int32_t* col_offsets_dev, void* stream, qg_packed_b** out) {
  if (!B_dev || !b_zp_host || !packed_dev || !col_offsets_dev || !out) return QG_ENULL;
  if (K <= 0 || N <= 0 || K > QG_MAX_K || ldb < (transposed ? K : N)) return QG_EINVAL;
  if (n_b_zp != 1 && n_b_zp != N) return QG_EINVAL;
  if (!aligned(packed_dev, 256) || !aligned(col_offsets_dev, 256)) return QG_EALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int K_pad = qg_round_up(K, QG_KPAD), N_pad = qg_round_up(N, QG_NPAD);

  qg_packed_b* h = new (std::nothrow) qg_packed_b();
  if (!h) return QG_ENOMEM;
  h->kind = QG_KIND_GEMM;
  h->version = QG_LAYOUT_VERSION;
  h->K = K;
  h->N = N;
  h->K_pad = K_pad;
  h->N_pad = N_pad;
  h->n_b_zp = n_b_zp;
  h->packed = static_cast<const int8_t*>(packed_dev);
  h->col_off = col_offsets_dev;
  h->bzp = col_offsets_dev + N_pad;
  h->G = h->R = h->S = h->Cg = h->Og = 0;
  h->conv_frags = nullptr;
  h->split = 0;
  h->frag_ptr = h->entries = nullptr;
  h->nnz = 0;

  int rc = upload_bzp(b_zp_host, n_b_zp, N, N_pad, col_offsets_dev + N_pad, s, &h->has_bzp);
  if (rc != QG_OK) {
    delete h;
    return rc;
  }
  if (qg_launch_pack_b(B_dev, K, N, ldb, transposed, K_pad, N_pad, static_cast<int8_t*>(packed_dev), col_offsets_dev,
                       col_offsets_dev + N_pad, s) != hipSuccess) {
    delete h;
    return QG_ELAUNCH;
  }
  *out = h;
  return QG_OK;
}

void qg_packed_b_destroy(qg_packed_b* p) { delete p; }

int qg_packed_b_k(const qg_packed_b* p) { return p ? p->K : 0; }
int qg_packed_b_n(const qg_packed_b* p) { return p ? p->N : 0; }

int qg_count_outliers(const int8_t* B_dev, int K, int N, int ldb, void* scratch_dev, size_t* nnz_host, void* stream) {
  if (!B_dev || !scratch_dev || !nnz_host) return QG_ENULL;
  if (K <= 0 || N <= 0 || K > QG_MAX_K || ldb < N) return QG_EINVAL;
  if (!aligned(scratch_dev, 8)) return QG_EALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  unsigned long long* cnt = static_cast<unsigned long long*>(scratch_dev);
  if (qg_launch_count_outliers(B_dev, K, N, ldb, cnt, s) != hipSuccess) return QG_ELAUNCH;
  unsigned long long host = 0;
  if (hipMemcpyAsync(&host, cnt, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess) return QG_ELAUNCH;
  if (hipStreamSynchronize(s) != hipSuccess) return QG_ELAUNCH;
  *nnz_host = (size_t)host;
  return QG_OK;
}

// [frag_ptr: nbucket+1][cursor: nbucket] int32, rounded up to 256 B; one bucket per fragment of the packed matrix
static size_t sparse_buckets(int K_pad, int N_pad) { return (size_t)(N_pad / QG_FRAG_COLS) * (size_t)(K_pad / QG_FRAG_K); }
static size_t sparse_header_bytes(int K_pad, int N_pad) {
  return ((2 * sparse_buckets(K_pad, N_pad) + 1) * sizeof(int32_t) + 255) / 256 * 256;
}

int qg_pack_b_outlier_sizes(int K, int N, size_t max_nnz, size_t* packed_bytes, size_t* col_offsets_bytes,
                            size_t* sparse_bytes) {
  if (!packed_bytes || !col_offsets_bytes || !sparse_bytes) return QG_ENULL;
  if (K <= 0 || N <= 0 || K > QG_MAX_K) return QG_EINVAL;
  if (max_nnz > (size_t)0x7FFFFFFF) return QG_EINVAL;
  const size_t K_pad = (size_t)qg_round_up(K, QG_KPAD), N_pad = (size_t)qg_round_up(N, QG_NPAD);
  *packed_bytes = K_pad * N_pad / 2;
  *col_offsets_bytes = 2 * N_pad * sizeof(int32_t);
  *sparse_bytes = sparse_header_bytes((int)K_pad, (int)N_pad) + (max_nnz ? max_nnz : 1) * sizeof(int32_t);
  return QG_OK;
}

int qg_pack_b_outlier(const int8_t* B_dev, int K, int N, int ldb, const int32_t* b_zp_host, int n_b_zp,
                      size_t max_nnz, void* packed_dev, int32_t* col_offsets_dev, void* sparse_dev, void* stream,
                      qg_packed_b** out) {
  if (!B_dev || !b_zp_host || !packed_dev || !col_offsets_dev || !sparse_dev || !out) return QG_ENULL;
  if (K <= 0 || N <= 0 || K > QG_MAX_K || ldb < N) return QG_EINVAL;
  if (n_b_zp != 1 && n_b_zp != N) return QG_EINVAL;
  if (max_nnz > (size_t)0x7FFFFFFF) return QG_EINVAL;
  if (!aligned(packed_dev, 256) || !aligned(col_offsets_dev, 256) || !aligned(sparse_dev, 256)) return QG_EALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int K_pad = qg_round_up(K, QG_KPAD), N_pad = qg_round_up(N, QG_NPAD);
  const size_t nbucket = sparse_buckets(K_pad, N_pad);
  int32_t* frag_ptr = static_cast<int32_t*>(sparse_dev);
  int32_t* cursor = frag_ptr + nbucket + 1;
  int32_t* entries =
      reinterpret_cast<int32_t*>(static_cast<unsigned char*>(sparse_dev) + sparse_header_bytes(K_pad, N_pad));

  qg_packed_b* h = new (std::nothrow) qg_packed_b();
  if (!h) return QG_ENOMEM;
  h->kind = QG_KIND_GEMM;
  h->version = QG_LAYOUT_VERSION;
  h->K = K;
  h->N = N;
  h->K_pad = K_pad;
  h->N_pad = N_pad;
  h->n_b_zp = n_b_zp;
  h->packed = static_cast<const int8_t*>(packed_dev);
  h->col_off = col_offsets_dev;
  h->bzp = col_offsets_dev + N_pad;
  h->G = h->R = h->S = h->Cg = h->Og = 0;
  h->conv_frags = nullptr;
  h->split = 1;
  h->frag_ptr = frag_ptr;
  h->entries = entries;
  h->nnz = 0;

  int rc = upload_bzp(b_zp_host, n_b_zp, N, N_pad, col_offsets_dev + N_pad, s, &h->has_bzp);
  int32_t total = 0;
  if (rc == QG_OK && qg_launch_pack_b_split_count(B_dev, K, N, ldb, K_pad, N_pad, static_cast<uint8_t*>(packed_dev),
                                                  col_offsets_dev, col_offsets_dev + N_pad, frag_ptr, cursor,
                                                  s) != hipSuccess)
    rc = QG_ELAUNCH;
  // the total decides whether the fill may run: it must not write past the caller's capacity
  if (rc == QG_OK && (hipMemcpyAsync(&total, frag_ptr + nbucket, sizeof(total), hipMemcpyDeviceToHost, s) != hipSuccess ||
                      hipStreamSynchronize(s) != hipSuccess))
    rc = QG_ELAUNCH;
  if (rc == QG_OK && (total < 0 || (size_t)total > max_nnz)) rc = QG_ECAPACITY;
  if (rc == QG_OK && total > 0 &&
      qg_launch_pack_b_split_fill(B_dev, K, N, ldb, K_pad, frag_ptr, cursor, entries, s) != hipSuccess)
    rc = QG_ELAUNCH;
  if (rc != QG_OK) {
    delete h;
    return rc;
  }
  h->nnz = total;
  *out = h;
  return QG_OK;
}

size_t qg_packed_b_nnz(const qg_packed_b* p) { return (p && p->split) ? (size_t)p->nnz : 0; }

size_t qg_gemm_workspace_bytes(int M, const qg_packed_b* Bp) {
  if (!Bp || M <= 0 || Bp->kind != QG_KIND_GEMM) return 0;
  int kernel = QG_KERNEL_AUTO;
  if (resolve_kernel(Bp, M, &kernel) != QG_OK) return 0;
  const int s = auto_ksplit(kernel, M, Bp);
  return s > 1 ? splitk_ws(kernel, M, Bp->N, s).bytes() : 0;
}

size_t qg_gemm_splitk_workspace_bytes(int M, const qg_packed_b* Bp, int kernel, int ksplit) {
  if (!Bp || M <= 0 || Bp->kind != QG_KIND_GEMM || ksplit < 0 || ksplit > kMaxKsplit) return 0;
  if (resolve_kernel(Bp, M, &kernel) != QG_OK) return 0;
  if (kernel == QG_KERNEL_TILE128) {
    const int s = ksplit > 1 ? clamp_ksplit_tile128(Bp, ksplit) : 1;
    return s > 1 ? splitk_ws(kernel, M, Bp->N, s).bytes() : 0;
  }
  if (kernel > QG_KERNEL_SKINNY64) return 0;
  const int s = ksplit == 0 ? auto_ksplit(kernel, M, Bp) : clamp_ksplit(Bp, ksplit);
  return s > 1 ? splitk_ws(kernel, M, Bp->N, s).bytes() : 0;
}

int qg_gemm_splitk_factor(int M, const qg_packed_b* Bp, int kernel, int ksplit) {
  if (!Bp || Bp->kind != QG_KIND_GEMM) return QG_ENULL;
  if (M <= 0 || ksplit < 0 || ksplit > kMaxKsplit) return QG_EINVAL;
  const int rc = resolve_kernel(Bp, M, &kernel);
  if (rc != QG_OK) return rc;
  if (kernel == QG_KERNEL_TILE128) return ksplit > 1 ? clamp_ksplit_tile128(Bp, ksplit) : 1;
  if (kernel > QG_KERNEL_SKINNY64) return 1;
  return ksplit == 0 ? auto_ksplit(kernel, M, Bp) : clamp_ksplit(Bp, ksplit);
}

int qg_gemm_workspace_init(void* workspace_dev, size_t bytes, void* stream) {
  if (bytes == 0) return QG_OK;
  if (!workspace_dev) return QG_ENULL;
  if (!aligned(workspace_dev, 16) || bytes % 4 != 0) return QG_EALIGN;
  const size_t n = bytes / 4;
  const unsigned blocks = (unsigned)((n + 255) / 256 < 2048 ? (n + 255) / 256 : 2048);
  hipLaunchKernelGGL(qg_fill_zero_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(stream),
                     static_cast<int32_t*>(workspace_dev), n);
  return hipGetLastError() == hipSuccess ? QG_OK : QG_ELAUNCH;
}

static int gemm_common(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp, qg_gemm_args* a) {
  if (!Bp || (!A_dev && M != 0)) return QG_ENULL;  // the data pointers of an empty batch are not referenced
  if (Bp->kind != QG_KIND_GEMM || Bp->version != QG_LAYOUT_VERSION) return QG_EINVAL;
  if (M < 0 || lda < Bp->K) return QG_EINVAL;
  a->A = A_dev;
  a->Bp = Bp->packed;
  a->col_off = Bp->col_off;
  a->bzp = Bp->bzp;
  a->M = M;
  a->N = Bp->N;
  a->K = Bp->K;
  a->kb64 = Bp->K_pad / QG_FRAG_K;
  a->nb16 = Bp->N_pad / QG_FRAG_COLS;
  a->has_bzp = Bp->has_bzp;
  a->sp_ptr = Bp->split ? Bp->frag_ptr : nullptr;
  a->sp_entries = Bp->entries;
  a->sp_total = (int)Bp->nnz;
  a->lda = lda;
  a->ksplit = 1;
  a->ks_per = a->kb64;
  return QG_OK;
}

static int gemm_requant(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp, const qg_requant_params* p,
                        uint8_t* C_dev, int ldc, void* workspace_dev, size_t workspace_bytes, bool bytes_known,
                        void* stream, int kernel, int ksplit) {
  qg_gemm_args a = {};
  int rc = gemm_common(A_dev, M, lda, Bp, &a);
  if (rc != QG_OK) return rc;
  rc = resolve_call(Bp, M, &kernel, &ksplit, {a_align(A_dev, lda), u8_kind(C_dev, ldc), Bp->has_bzp != 0}, workspace_dev);
  if (rc != QG_OK) return rc;
  if (!C_dev && M != 0) return QG_ENULL;
  rc = check_requant(p, Bp->N);
  if (rc != QG_OK) return rc;
  if (ldc < Bp->N) return QG_EINVAL;
  rc = resolve_ksplit(Bp, M, kernel, ksplit, workspace_dev, workspace_bytes, bytes_known, &a);
  if (rc != QG_OK) return rc;
  a.bias = p->bias;
  a.scales = p->scales;
  a.scale_stride = p->n_scales == 1 ? 0 : 1;
  a.a_zp_m128 = p->a_zp - 128;
  a.c_zp = p->c_zp;
  const int lo = p->relu ? p->c_zp : 0;
  a.clamp_lo = (float)(lo - p->c_zp);
  a.clamp_hi = (float)(255 - p->c_zp);
  a.C = C_dev;
  a.ldc = ldc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // 4-byte stores in the streaming kernels, 16-byte stores in the tiled ones
  a.c_vec = kernel <= QG_KERNEL_SKINNY64 ? (aligned(C_dev, 4) && (ldc % 4 == 0)) : (aligned(C_dev, 16) && (ldc % 16 == 0));
  a.c_wt = (long long)M * Bp->N <= (1 << 18);
  if (M == 0) return QG_OK;  // an empty batch: checked like any other, nothing to enqueue
  const hipError_t e = launch_gemm(a, QG_MODE_REQUANT, kernel, s);
  return e == hipSuccess ? QG_OK : QG_ELAUNCH;
}

int qg_gemm_u8s8_requant(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp,
                         const qg_requant_params* p, uint8_t* C_dev, int ldc, void* workspace_dev,
                         void* stream) {
  return gemm_requant(A_dev, M, lda, Bp, p, C_dev, ldc, workspace_dev, 0, false, stream, QG_KERNEL_AUTO, 0);
}

int qg_gemm_u8s8_requant_kernel(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp,
                                const qg_requant_params* p, uint8_t* C_dev, int ldc, void* workspace_dev,
                                void* stream, int kernel) {
  return gemm_requant(A_dev, M, lda, Bp, p, C_dev, ldc, workspace_dev, 0, false, stream, kernel, 0);
}

int qg_gemm_u8s8_requant_splitk(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp,
                                const qg_requant_params* p, uint8_t* C_dev, int ldc, void* workspace_dev,
                                size_t workspace_bytes, void* stream, int kernel, int ksplit) {
  return gemm_requant(A_dev, M, lda, Bp, p, C_dev, ldc, workspace_dev, workspace_bytes, true, stream, kernel, ksplit);
}

int qg_gemm_u8s8_requant_noalloc(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp,
                                 const qg_requant_params* p, uint8_t* C_dev, int ldc, void* stream, int kernel,
                                 int ksplit) {
  if (!Bp) return QG_ENULL;
  if (Bp->kind != QG_KIND_GEMM || Bp->version != QG_LAYOUT_VERSION || M < 0) return QG_EINVAL;
  // the split this call would use with a workspace at hand, and what it needs of the built-in scratch
  const size_t need = M > 0 ? qg_gemm_splitk_workspace_bytes(M, Bp, kernel, ksplit) : 0;
  if (need > QG_NOALLOC_SCRATCH_BYTES) return QG_EWORKSPACE;
  void* scratch = nullptr;
  const int rc = noalloc_scratch(&scratch);
  if (rc != QG_OK) return rc;
  return gemm_requant(A_dev, M, lda, Bp, p, C_dev, ldc, scratch, QG_NOALLOC_SCRATCH_BYTES, true, stream, kernel, ksplit);
}

static int gemm_acc32(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp, int32_t* C32_dev, int ldc,
                      int32_t* rowsum_dev, void* workspace_dev, size_t workspace_bytes, bool bytes_known, void* stream,
                      int kernel, int ksplit) {
  qg_gemm_args a = {};
  int rc = gemm_common(A_dev, M, lda, Bp, &a);
  if (rc != QG_OK) return rc;
  rc = resolve_call(Bp, M, &kernel, &ksplit, {a_align(A_dev, lda), OUT_I32, Bp->has_bzp != 0}, workspace_dev);
  if (rc != QG_OK) return rc;
  if (!C32_dev && M != 0) return QG_ENULL;
  if (ldc < Bp->N) return QG_EINVAL;
  rc = resolve_ksplit(Bp, M, kernel, ksplit, workspace_dev, workspace_bytes, bytes_known, &a);
  if (rc != QG_OK) return rc;
  a.C32 = C32_dev;
  a.rowsum_out = rowsum_dev;
  a.ldc = ldc;
  if (M == 0) return QG_OK;
  const hipError_t e = launch_gemm(a, QG_MODE_ACC32, kernel, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? QG_OK : QG_ELAUNCH;
}

int qg_gemm_u8s8_acc32(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp, int32_t* C32_dev,
                       int ldc, int32_t* rowsum_dev, void* workspace_dev, void* stream) {
  return gemm_acc32(A_dev, M, lda, Bp, C32_dev, ldc, rowsum_dev, workspace_dev, 0, false, stream, QG_KERNEL_AUTO, 0);
}

int qg_gemm_u8s8_acc32_kernel(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp, int32_t* C32_dev,
                              int ldc, int32_t* rowsum_dev, void* workspace_dev, void* stream, int kernel) {
  return gemm_acc32(A_dev, M, lda, Bp, C32_dev, ldc, rowsum_dev, workspace_dev, 0, false, stream, kernel, 0);
}

int qg_gemm_u8s8_acc32_splitk(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp, int32_t* C32_dev,
                              int ldc, int32_t* rowsum_dev, void* workspace_dev, size_t workspace_bytes, void* stream,
                              int kernel, int ksplit) {
  return gemm_acc32(A_dev, M, lda, Bp, C32_dev, ldc, rowsum_dev, workspace_dev, workspace_bytes, true, stream, kernel,
                    ksplit);
}

static int check_dequant(const qg_dequant_params* p, int N) {
  if (!p) return QG_ENULL;
  if (!p->scales) return QG_ENULL;
  if (p->a_zp < 0 || p->a_zp > 255) return QG_EINVAL;
  if (p->n_scales != 1 && p->n_scales != N) return QG_EINVAL;
  if (p->relu != 0 && p->relu != 1) return QG_EINVAL;
  return QG_OK;
}

int qg_gemm_u8s8_dequant_f32(const uint8_t* A_dev, int M, int lda, const qg_packed_b* Bp,
                             const qg_dequant_params* p, float* C_dev, int ldc, void* workspace_dev,
                             void* stream, int kernel) {
  qg_gemm_args a = {};
  int rc = gemm_common(A_dev, M, lda, Bp, &a);
  if (rc != QG_OK) return rc;
  int ksplit = 0;
  rc = resolve_call(Bp, M, &kernel, &ksplit, {a_align(A_dev, lda), OUT_F32, Bp->has_bzp != 0}, workspace_dev);
  if (rc != QG_OK) return rc;
  if (!C_dev && M != 0) return QG_ENULL;
  rc = check_dequant(p, Bp->N);
  if (rc != QG_OK) return rc;
  if (ldc < Bp->N) return QG_EINVAL;
  if (!aligned(C_dev, 4)) return QG_EALIGN;
  rc = resolve_ksplit(Bp, M, kernel, ksplit, workspace_dev, 0, false, &a);
  if (rc != QG_OK) return rc;
  a.bias = p->bias;
  a.scales = p->scales;
  a.scale_stride = p->n_scales == 1 ? 0 : 1;
  a.a_zp_m128 = p->a_zp - 128;
  a.relu_lo = p->relu ? 0.0f : -INFINITY;
  a.Cf = C_dev;
  a.ldc = ldc;
  a.c_vec = aligned(C_dev, 16) && (ldc % 4 == 0);
  if (M == 0) return QG_OK;
  const hipError_t e = launch_gemm(a, QG_MODE_DEQUANT, kernel, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? QG_OK : QG_ELAUNCH;
}

int qg_quantize_a_f32(const float* A_dev, int M, int K, int lda, float inv_scale, int a_zp, uint8_t* Aq_dev,
                      int ldq, void* stream) {
  if ((!A_dev || !Aq_dev) && M != 0) return QG_ENULL;
  if (M < 0 || K <= 0 || lda < K || ldq < K) return QG_EINVAL;
  if (a_zp < 0 || a_zp > 255 || !(inv_scale > 0.0f) || !isfinite(inv_scale)) return QG_EINVAL;
  if (!aligned(A_dev, 4)) return QG_EALIGN;
  if (M == 0) return QG_OK;
  const hipError_t e =
      qg_launch_quantize_a(A_dev, M, K, lda, inv_scale, a_zp, Aq_dev, ldq, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? QG_OK : QG_ELAUNCH;
}

// row pitch of the quantized copy in the workspace: whole 16-byte chunks, so the copy takes the vector paths
static int f32_ldq(const qg_packed_b* Bp) { return qg_round_up(Bp->K, 16); }

size_t qg_gemm_f32_workspace_bytes(int M, const qg_packed_b* Bp) {
  if (!Bp || M <= 0 || Bp->kind != QG_KIND_GEMM) return 0;
  return (size_t)M * (size_t)f32_ldq(Bp);  // what a tiled kernel needs; a streaming kernel needs none
}

// whether rows of the fp32 A share memory with rows of C
static bool f32_in_place(const float* A_dev, int M, int lda, int K, const void* C_dev, int ldc, int N, size_t c_size) {
  if (M <= 0) return false;
  const uintptr_t a = reinterpret_cast<uintptr_t>(A_dev), c = reinterpret_cast<uintptr_t>(C_dev);
  return a < c + ((size_t)(M - 1) * ldc + N) * c_size && c < a + ((size_t)(M - 1) * lda + K) * sizeof(float);
}

// With a workspace: the kernel of an automatic call, and whether it quantizes A itself.  Not where C lies over A: the two launches
// have read all of A before they write C, in one launch every column block reads A while others already write.
static int f32_resolve(const qg_packed_b* Bp, int M, int* kernel, bool* one_launch, const call_form& f, bool in_place) {
  if (*kernel == QG_KERNEL_AUTO && !in_place && !Bp->split && M > 0 && rule_kernel(M, Bp->N, Bp->K) == QG_KERNEL_AUTO) {
    const int k = f32_select(M, Bp->N, Bp->K, f);
    if (k != QG_KERNEL_AUTO) {
      *kernel = k;
      *one_launch = true;
      return QG_OK;
    }
  }
  int ksplit = 1;
  return resolve_call(Bp, M, kernel, &ksplit, f, nullptr);
}

// Without a workspace: whether one launch serves the call is builtin_select's answer, whatever the call's form (tiled kernels need the
// workspace), and where it does, the streaming kernel goes by the prices above.
static int f32_resolve_alone(const qg_packed_b* Bp, int M, int* kernel, const call_form& f) {
  const bool choose = *kernel == QG_KERNEL_AUTO && !Bp->split && M > 0 && M <= k_f32_most_rows && rule_kernel(M, Bp->N, Bp->K) == QG_KERNEL_AUTO;
  const int rc = resolve_kernel(Bp, M, kernel);
  if (rc == QG_OK && choose && *kernel <= QG_KERNEL_SKINNY64) *kernel = f32_one_launch(M, Bp->N, Bp->K, f, 1e300);
  return rc;
}

static int quantize_into_workspace(const float* A_dev, int M, int lda, float a_inv_scale, const qg_packed_b* Bp,
                                   int a_zp, void* workspace_dev, void* stream) {
  if (!Bp || (!A_dev && M != 0)) return QG_ENULL;
  if (Bp->kind != QG_KIND_GEMM || Bp->version != QG_LAYOUT_VERSION) return QG_EINVAL;
  if (M == 0)  // an empty batch needs no workspace; the remaining arguments are still checked
    return (lda < Bp->K || a_zp < 0 || a_zp > 255 || !(a_inv_scale > 0.0f) || !isfinite(a_inv_scale)) ? QG_EINVAL : QG_OK;
  if (!workspace_dev) return QG_EWORKSPACE;
  if (!aligned(workspace_dev, 16)) return QG_EALIGN;
  return qg_quantize_a_f32(A_dev, M, Bp->K, lda, a_inv_scale, a_zp, static_cast<uint8_t*>(workspace_dev),
                           f32_ldq(Bp), stream);
}

// fp32 activations on a streaming kernel: ONE launch -- the kernel quantizes the block it stages (Appendix B: any packing routine
// for A; row offsets come from the staged block in the same pass) and, where there is a workspace, leaves the quantized rows there
// as the separate pass does.  For a caller without a workspace whatever streaming kernel is in use; with one where QG_KERNEL_AUTO
// finds it faster (`one_launch`: 16 x 512 x 512 4.6 us in two launches, 3.8 so; 16 x 4096 x 4096, 5.6 in two and 6.7 so, stays in two, and so does
// 512 x 4096 x 4096).  Fills the common fields of `a`; returns QG_OK with *fused = false for two launches.
static int f32_fused_common(const float* A_dev, int M, int lda, float a_inv_scale, int a_zp, const qg_packed_b* Bp,
                            int kernel, bool one_launch, void* workspace_dev, qg_gemm_args* a, bool* fused) {
  *fused = false;
  if (kernel > QG_KERNEL_SKINNY64 || Bp->split || (workspace_dev != nullptr && !one_launch)) return QG_OK;
  if (!A_dev && M != 0) return QG_ENULL;
  if (workspace_dev != nullptr && !aligned(workspace_dev, 16)) return QG_EALIGN;
  if (lda < Bp->K || a_zp < 0 || a_zp > 255 || !(a_inv_scale > 0.0f) || !isfinite(a_inv_scale)) return QG_EINVAL;
  if (!aligned(A_dev, 4)) return QG_EALIGN;
  int rc = gemm_common(reinterpret_cast<const uint8_t*>(A_dev), M, lda, Bp, a);
  if (rc != QG_OK) return rc;
  a->q_inv = a_inv_scale;
  a->q_zp = (float)a_zp;
  a->q_copy = static_cast<uint8_t*>(workspace_dev);
  a->q_ldq = f32_ldq(Bp);
  *fused = true;
  return QG_OK;
}

int qg_gemm_f32s8_requant(const float* A_dev, int M, int lda, float a_inv_scale, const qg_packed_b* Bp,
                          const qg_requant_params* p, uint8_t* C_dev, int ldc, void* workspace_dev,
                          void* stream, int kernel) {
  // every check of the second stage first, so that an error leaves nothing enqueued
  if (!Bp || !p || (!C_dev && M != 0)) return QG_ENULL;
  if (Bp->kind != QG_KIND_GEMM || Bp->version != QG_LAYOUT_VERSION) return QG_EINVAL;
  int rc = check_requant(p, Bp->N);
  if (rc != QG_OK) return rc;
  if (M < 0 || ldc < Bp->N) return QG_EINVAL;
  // (with a workspace the 8-bit call below runs on the quantized copy, whose rows are 16-byte aligned and which has no split)
  bool one_launch = false;
  rc = workspace_dev ? f32_resolve(Bp, M, &kernel, &one_launch, {16, u8_kind(C_dev, ldc), Bp->has_bzp != 0},
                                 f32_in_place(A_dev, M, lda, Bp->K, C_dev, ldc, Bp->N, 1))
                     : f32_resolve_alone(Bp, M, &kernel, {16, u8_kind(C_dev, ldc), Bp->has_bzp != 0});
  if (rc != QG_OK) return rc;
  {
    qg_gemm_args a = {};
    bool fused = false;
    rc = f32_fused_common(A_dev, M, lda, a_inv_scale, p->a_zp, Bp, kernel, one_launch, workspace_dev, &a, &fused);
    if (rc != QG_OK) return rc;
    if (fused) {
      a.bias = p->bias;
      a.scales = p->scales;
      a.scale_stride = p->n_scales == 1 ? 0 : 1;
      a.a_zp_m128 = p->a_zp - 128;
      a.c_zp = p->c_zp;
      const int lo = p->relu ? p->c_zp : 0;
      a.clamp_lo = (float)(lo - p->c_zp);
      a.clamp_hi = (float)(255 - p->c_zp);
      a.C = C_dev;
      a.ldc = ldc;
      a.c_vec = aligned(C_dev, 4) && (ldc % 4 == 0);
      a.c_wt = (long long)M * Bp->N <= (1 << 18);
      if (M == 0) return QG_OK;
      const hipError_t e = qg_launch_gemm_skinny_f32(a, QG_MODE_REQUANT, kernel, static_cast<hipStream_t>(stream));
      return e == hipSuccess ? QG_OK : QG_ELAUNCH;
    }
  }
  rc = quantize_into_workspace(A_dev, M, lda, a_inv_scale, Bp, p->a_zp, workspace_dev, stream);
  if (rc != QG_OK || M == 0) return rc;
  return qg_gemm_u8s8_requant_kernel(static_cast<const uint8_t*>(workspace_dev), M, f32_ldq(Bp), Bp, p, C_dev, ldc,
                                     nullptr, stream, kernel);
}

int qg_gemm_f32s8_dequant_f32(const float* A_dev, int M, int lda, float a_inv_scale, const qg_packed_b* Bp,
                              const qg_dequant_params* p, float* C_dev, int ldc, void* workspace_dev,
                              void* stream, int kernel) {
  if (!Bp || !p || (!C_dev && M != 0)) return QG_ENULL;
  if (Bp->kind != QG_KIND_GEMM || Bp->version != QG_LAYOUT_VERSION) return QG_EINVAL;
  int rc = check_dequant(p, Bp->N);
  if (rc != QG_OK) return rc;
  if (M < 0 || ldc < Bp->N) return QG_EINVAL;
  bool one_launch = false;
  rc = workspace_dev ? f32_resolve(Bp, M, &kernel, &one_launch, {16, OUT_F32, Bp->has_bzp != 0},
                                   f32_in_place(A_dev, M, lda, Bp->K, C_dev, ldc, Bp->N, sizeof(float)))
                     : f32_resolve_alone(Bp, M, &kernel, {16, OUT_F32, Bp->has_bzp != 0});
  if (rc != QG_OK) return rc;
  if (!aligned(C_dev, 4)) return QG_EALIGN;
  {
    qg_gemm_args a = {};
    bool fused = false;
    rc = f32_fused_common(A_dev, M, lda, a_inv_scale, p->a_zp, Bp, kernel, one_launch, workspace_dev, &a, &fused);
    if (rc != QG_OK) return rc;
    if (fused) {
      a.bias = p->bias;
      a.scales = p->scales;
      a.scale_stride = p->n_scales == 1 ? 0 : 1;
      a.a_zp_m128 = p->a_zp - 128;
      a.relu_lo = p->relu ? 0.0f : -INFINITY;
      a.Cf = C_dev;
      a.ldc = ldc;
      a.c_vec = aligned(C_dev, 16) && (ldc % 4 == 0);
      if (M == 0) return QG_OK;
      const hipError_t e = qg_launch_gemm_skinny_f32(a, QG_MODE_DEQUANT, kernel, static_cast<hipStream_t>(stream));
      return e == hipSuccess ? QG_OK : QG_ELAUNCH;
    }
  }
  rc = quantize_into_workspace(A_dev, M, lda, a_inv_scale, Bp, p->a_zp, workspace_dev, stream);
  if (rc != QG_OK || M == 0) return rc;
  return qg_gemm_u8s8_dequant_f32(static_cast<const uint8_t*>(workspace_dev), M, f32_ldq(Bp), Bp, p, C_dev, ldc,
                                  nullptr, stream, kernel);
}

namespace {
// One convolution as a GEMM with the im2col folded into the requests: Cin channels starting at `in` of pixels that
// are `pix` bytes apart (a whole image, or the channel slice of one group), weights as a packed K x N matrix with
// K = R*S*Cin; output channel j goes to out[pixel * ldc + j]; bias and scales (when per channel) start at entry ch0.
int launch_conv_gemm(const uint8_t* in, int in_bytes, int Nb, int H, int W, int Cin, int pix, int R, int S, int pad, int stride,
                     int Ho, int Wo, const int8_t* packed, const int32_t* col_off, const int32_t* bzp, int K, int K_pad, int N,
                     int N_pad, int has_bzp, const qg_requant_params* p, int ch0, uint8_t* out, int ldc, int kernel,
                     hipStream_t stream) {
  qg_gemm_args a = {};
  a.A = in;
  a.Bp = packed;
  a.col_off = col_off;
  a.bzp = bzp;
  a.M = Nb * Ho * Wo;
  a.N = N;
  a.K = K;
  a.kb64 = K_pad / QG_FRAG_K;
  a.nb16 = N_pad / QG_FRAG_COLS;
  a.has_bzp = has_bzp;
  a.lda = 0;
  a.bias = p->bias ? p->bias + ch0 : nullptr;
  a.scales = p->n_scales == 1 ? p->scales : p->scales + ch0;
  a.scale_stride = p->n_scales == 1 ? 0 : 1;
  a.a_zp_m128 = p->a_zp - 128;
  a.c_zp = p->c_zp;
  const int lo = p->relu ? p->c_zp : 0;
  a.clamp_lo = (float)(lo - p->c_zp);
  a.clamp_hi = (float)(255 - p->c_zp);
  a.C = out;
  a.ldc = ldc;
  a.c_vec = aligned(out, 16) && (ldc % 16 == 0);
  a.cv_H = H;
  a.cv_W = W;
  a.cv_Cin = Cin;
  a.cv_pix = pix;
  a.cv_Ho = Ho;
  a.cv_Wo = Wo;
  a.cv_R = R;
  a.cv_S = S;
  a.cv_stride = stride;
  a.cv_pad = pad;
  a.cv_azp = p->a_zp;
  a.cv_in_bytes = in_bytes;
  // the tiled kernels, chosen by the same cost formula as a GEMM's; few pixels and a long K go to the 16-row streaming
  // kernel where it applies (at most 32 taps), priced with the streaming formula and the constants measured for the
  // convolution's requests
  const bool stream_ok = Cin % 16 == 0 && R * S <= 32;  // (asked for by id they take whole 64-channel slices only, as ever)
  const bool explicit_kernel = kernel != QG_KERNEL_AUTO;
  if (!explicit_kernel) {
    double best_us = 1e300;
    for (const conv_tile_price& c : k_conv_tile_price) {
      const double us = conv_tile_us(c, a);
      if (us < best_us) best_us = us, kernel = c.kernel;
    }
    for (const conv_patch_price& c : k_conv_patch_price) {
      const int per_cu = qg_conv_patch_per_cu(a, c.kernel - QG_KERNEL_PATCH64X128);
      if (per_cu == 0) continue;
      const int sets = c.kernel == QG_KERNEL_PATCH64X128 ? qg_conv_patch_sets(a) : 0;
      const double us = conv_patch_us(sets == 4 ? k_conv_few4_price : sets == 2 ? k_conv_few2_price : c, a, per_cu);
      if (us < best_us) best_us = us, kernel = c.kernel;
    }
    if (stream_ok)
      for (int i = 0; i < (Cin % QG_FRAG_K == 0 ? 3 : 2); ++i) {  // (64 rows take whole k blocks per tap)
        const conv_stream_price& c = k_conv_stream_price[2 * i + (tiles_of(a.M, a.N, k_conv_stream_price[2 * i].rows, 32) > 128 ? 1 : 0)];
        const double us = conv_stream_us(c, a);
        if (ceil_div(a.M, c.rows) <= 65535 && us < best_us) best_us = us, kernel = c.kernel;
      }
  }
  if (kernel >= QG_KERNEL_PATCH64X128) {
    const int form = kernel - QG_KERNEL_PATCH64X128;
    if (!qg_conv_patch_applies(a, form)) return QG_EUNSUPPORTED;
    return qg_launch_conv_patch(a, form, stream) == hipSuccess ? QG_OK : QG_ELAUNCH;
  }
  if (kernel <= QG_KERNEL_SKINNY64) {
    if (!stream_ok || (explicit_kernel && Cin % QG_FRAG_K != 0)) return QG_EUNSUPPORTED;
    a.ksplit = 1;
    a.ks_per = a.kb64;
    a.c_vec = aligned(out, 4) && (ldc % 4 == 0);
    a.c_wt = (long long)a.M * N <= (1 << 18);
    const hipError_t e = qg_launch_conv_skinny(a, kernel, stream);
    return e == hipSuccess ? QG_OK : QG_ELAUNCH;
  }
  const hipError_t e = qg_launch_conv_dense(a, kernel, stream);
  return e == hipSuccess ? QG_OK : QG_ELAUNCH;
}
}  // namespace

int qg_conv_dense_u8s8_requant(const uint8_t* in_nhwc, int Nb, int H, int W, int Cin, int R, int S, int pad,
                               int stride, const qg_packed_b* Wp, const qg_requant_params* p, uint8_t* out_nhwc,
                               void* stream, int kernel) {
  if (!Wp || ((!in_nhwc || !out_nhwc) && Nb != 0)) return QG_ENULL;
  if (Wp->kind != QG_KIND_GEMM || Wp->version != QG_LAYOUT_VERSION) return QG_EINVAL;
  if (kernel < QG_KERNEL_AUTO || kernel > QG_KERNEL_CONV_LAST) return QG_EINVAL;
  if (kernel == QG_KERNEL_TILE256) return QG_EUNSUPPORTED;
  if (Nb < 0 || H <= 0 || W <= 0 || Cin <= 0 || R <= 0 || S <= 0 || pad < 0 || stride <= 0) return QG_EINVAL;
  if ((long long)R * S * Cin != Wp->K) return QG_EINVAL;
  int rc = check_requant(p, Wp->N);
  if (rc != QG_OK) return rc;
  if (H + 2 * pad < R || W + 2 * pad < S) return QG_EINVAL;
  const int Ho = (H + 2 * pad - R) / stride + 1, Wo = (W + 2 * pad - S) / stride + 1;
  if (Wp->split) return QG_EUNSUPPORTED;
  if (Cin % 16 != 0 || !aligned(in_nhwc, 16)) {
    // no staged kernel takes these extents: the byte-gathering kernel, under the automatic choice only
    if (kernel != QG_KERNEL_AUTO) return QG_EUNSUPPORTED;
    if ((uint64_t)Nb * H * W * Cin >= (1ull << 31) || (uint64_t)Nb * Ho * Wo * Wp->N >= (1ull << 31)) return QG_EUNSUPPORTED;
    qg_conv_args c = {};
    c.in = in_nhwc;
    c.Bp = Wp->packed;
    c.nb16 = Wp->N_pad / QG_FRAG_COLS;
    c.col_off = Wp->col_off;
    c.bzp = Wp->bzp;
    c.bias = p->bias;
    c.scales = p->scales;
    c.out = out_nhwc;
    c.Nb = Nb;
    c.H = H;
    c.W = W;
    c.C = Cin;
    c.Ho = Ho;
    c.Wo = Wo;
    c.Cout = Wp->N;
    c.G = 1;
    c.Cg = Cin;
    c.Og = Wp->N;
    c.R = R;
    c.S = S;
    c.pad = pad;
    c.stride = stride;
    c.scale_stride = p->n_scales == 1 ? 0 : 1;
    c.a_zp = p->a_zp;
    c.c_zp = p->c_zp;
    const int lo = p->relu ? p->c_zp : 0;
    c.clamp_lo = (float)(lo - p->c_zp);
    c.clamp_hi = (float)(255 - p->c_zp);
    c.has_bzp = Wp->has_bzp;
    if (Nb == 0) return QG_OK;
    const hipError_t e = qg_conv_runs_applies(c) ? qg_launch_conv_runs(c, static_cast<hipStream_t>(stream))
                                                 : qg_launch_conv_dense_plain(c, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? QG_OK : QG_ELAUNCH;
  }
  // 32-bit byte offsets into the image (tap offsets included) and 32-bit pixel counts
  if ((uint64_t)Nb * H * W * Cin >= (1ull << 30) || (uint64_t)Nb * Ho * Wo >= (1ull << 31) / 4) return QG_EUNSUPPORTED;
  // A 1 x 1 filter with unit stride and no padding is the plain GEMM over the pixel rows (lda = Cin): it takes
  // the GEMM's own kernels and choice, hand-scheduled loops included; the bytes are the same either way.
  if (R == 1 && S == 1 && pad == 0 && stride == 1) {
    if (kernel > QG_KERNEL_LAST) return QG_EUNSUPPORTED;  // the patch kernels have nothing to keep for a single tap
    return qg_gemm_u8s8_requant_kernel(in_nhwc, Nb * H * W, Cin, Wp, p, out_nhwc, Wp->N, nullptr, stream, kernel);
  }
  if (Nb == 0) return QG_OK;  // an empty batch
  return launch_conv_gemm(in_nhwc, Nb * H * W * Cin, Nb, H, W, Cin, Cin, R, S, pad, stride, Ho, Wo, Wp->packed, Wp->col_off,
                          Wp->bzp, Wp->K, Wp->K_pad, Wp->N, Wp->N_pad, Wp->has_bzp, p, 0, out_nhwc, Wp->N, kernel,
                          static_cast<hipStream_t>(stream));
}

namespace {
// the groups of 4 -> 4 channels with a 1 x 1 or 3 x 3 filter have a layout (and kernels) of their own
bool conv_is_4to4(int G, int R, int S, int Cg, int Og) {
  return Cg == 4 && Og == 4 && ((R == 1 && S == 1) || (R == 3 && S == 3)) && G <= 256;
}
// log2(Cg) when the block-diagonal matrix-core fragments exist for a general group shape (square groups of 1 -- a
// depthwise convolution --, 2, 8, 16 or 32 channels -- or of 4 in more than 256 groups --, 1 x 1 or 3 x 3, whole
// 32-channel blocks), else -1
int conv_mfma_lcg(int G, int R, int S, int Cg, int Og) {
  if (Cg != Og || !((R == 1 && S == 1) || (R == 3 && S == 3)) || (G * Cg) % 32 != 0) return -1;
  return Cg == 1 ? 0 : Cg == 2 ? 1 : Cg == 4 ? 2 : Cg == 8 ? 3 : Cg == 16 ? 4 : Cg == 32 ? 5 : -1;
}
// groups of a multiple of 16 channels without block-diagonal tiles: each group is a dense convolution of its own
// channel slice (one launch per group), with its weights packed as a GEMM matrix
bool conv_is_wide(int G, int R, int S, int Cg, int Og) {
  return !conv_is_4to4(G, R, S, Cg, Og) && conv_mfma_lcg(G, R, S, Cg, Og) < 0 && Cg % 16 == 0 && G <= 64;
}
}  // namespace

static int conv_sizes_without_gemms(int G, int R, int S, int Cg, int Og, size_t* packed_bytes, size_t* col_offsets_bytes);

int qg_pack_conv_w_sizes(int G, int R, int S, int Cg, int Og, size_t* packed_bytes,
                         size_t* col_offsets_bytes) {
  if (!packed_bytes || !col_offsets_bytes) return QG_ENULL;
  if (G <= 0 || R <= 0 || S <= 0 || Cg <= 0 || Og <= 0) return QG_EINVAL;
  if ((long long)R * S * Cg > QG_MAX_K || (long long)G * Cg >= (1 << 24) || (long long)G * Og >= (1 << 24)) return QG_EINVAL;
  const int rc = conv_sizes_without_gemms(G, R, S, Cg, Og, packed_bytes, col_offsets_bytes);
  if (rc != QG_OK) return rc;
  if (conv_is_wide(G, R, S, Cg, Og)) {
    const size_t kp = (size_t)qg_round_up(R * S * Cg, QG_KPAD), np = (size_t)qg_round_up(Og, QG_NPAD);
    *packed_bytes += (size_t)G * kp * np;
    *col_offsets_bytes += (size_t)G * 2 * np * sizeof(int32_t);
  }
  return QG_OK;
}

// the layouts every group shape has: the general (or 4 -> 4) weights, the block-diagonal tiles, the folded offsets
static int conv_sizes_without_gemms(int G, int R, int S, int Cg, int Og, size_t* packed_bytes, size_t* col_offsets_bytes) {
  if (conv_is_4to4(G, R, S, Cg, Og)) {
    // dot4 layout, then (when C = 4 G is a multiple of 32) the matrix-core fragments
    *packed_bytes = (size_t)qg_round_up(G * R * S * Cg * Og, 256) +
                    ((G % 8 == 0) ? (size_t)(G / 8) * R * S * QG_FRAG_BYTES : 0);
  } else {
    // general layout [Cout][R*S][Cg rounded up to 4], then the matrix-core fragments where they exist
    const size_t any = (size_t)G * Og * R * S * (size_t)qg_round_up(Cg, 4);
    if (any >= (1ull << 31)) return QG_EUNSUPPORTED;
    *packed_bytes = (any + 255) / 256 * 256 +
                    (conv_mfma_lcg(G, R, S, Cg, Og) >= 0 ? (size_t)(G * Cg / 32) * R * S * QG_FRAG_BYTES : 0);
  }
  *col_offsets_bytes = (size_t)qg_round_up(2 * G * Og * (int)sizeof(int32_t), 256);
  return QG_OK;
}

int qg_pack_conv_w(const int8_t* W_dev, int G, int R, int S, int Cg, int Og, const int32_t* b_zp_host,
                   int n_b_zp, void* packed_dev, int32_t* col_offsets_dev, void* stream,
                   qg_packed_b** out) {
  if (!W_dev || !b_zp_host || !packed_dev || !col_offsets_dev || !out) return QG_ENULL;
  size_t pb, cb;
  int rc = qg_pack_conv_w_sizes(G, R, S, Cg, Og, &pb, &cb);
  if (rc != QG_OK) return rc;
  const int Cout = G * Og;
  if (n_b_zp != 1 && n_b_zp != Cout) return QG_EINVAL;
  if (!aligned(packed_dev, 256) || !aligned(col_offsets_dev, 256)) return QG_EALIGN;
  hipStream_t s = static_cast<hipStream_t>(stream);
  qg_packed_b* h = new (std::nothrow) qg_packed_b();
  if (!h) return QG_ENOMEM;
  h->kind = QG_KIND_CONV;
  h->version = QG_LAYOUT_VERSION;
  h->K = R * S * Cg;
  h->N = Cout;
  h->K_pad = h->K;
  h->N_pad = Cout;
  h->n_b_zp = n_b_zp;
  h->packed = static_cast<const int8_t*>(packed_dev);
  h->col_off = col_offsets_dev;
  h->bzp = col_offsets_dev + Cout;
  h->G = G;
  h->R = R;
  h->S = S;
  h->Cg = Cg;
  h->Og = Og;
  h->split = 0;
  h->frag_ptr = h->entries = nullptr;
  h->nnz = 0;
  const bool four = conv_is_4to4(G, R, S, Cg, Og);
  const int lcg = four ? 2 : conv_mfma_lcg(G, R, S, Cg, Og);
  int8_t* frags = nullptr;
  if (four)
    frags = (G % 8 == 0) ? static_cast<int8_t*>(packed_dev) + qg_round_up(G * R * S * Cg * Og, 256) : nullptr;
  else if (lcg >= 0)
    frags = static_cast<int8_t*>(packed_dev) + ((size_t)Cout * R * S * (size_t)qg_round_up(Cg, 4) + 255) / 256 * 256;
  h->conv_frags = frags;
  h->conv_any = four ? nullptr : static_cast<const int8_t*>(packed_dev);
  rc = upload_bzp(b_zp_host, n_b_zp, Cout, Cout, col_offsets_dev + Cout, s, &h->has_bzp);
  if (rc != QG_OK) {
    delete h;
    return rc;
  }
  const hipError_t e = four ? qg_launch_pack_conv_w(W_dev, G, R * S, static_cast<int8_t*>(packed_dev), col_offsets_dev,
                                                    col_offsets_dev + Cout, frags, s)
                            : qg_launch_pack_conv_w_any(W_dev, G, R * S, Cg, Og, static_cast<int8_t*>(packed_dev),
                                                        col_offsets_dev, col_offsets_dev + Cout, frags, lcg, s);
  if (e != hipSuccess) {
    delete h;
    return QG_ELAUNCH;
  }
  h->conv_gemm = nullptr;
  h->conv_gemm_off = nullptr;
  if (conv_is_wide(G, R, S, Cg, Og)) {
    const int K = R * S * Cg, kp = qg_round_up(K, QG_KPAD), np = qg_round_up(Og, QG_NPAD);
    size_t pb0, cb0;
    conv_sizes_without_gemms(G, R, S, Cg, Og, &pb0, &cb0);
    int8_t* gp = static_cast<int8_t*>(packed_dev) + pb0;
    int32_t* go = col_offsets_dev + cb0 / sizeof(int32_t);
    for (int g = 0; g < G; ++g) {
      int unused;
      rc = upload_bzp(n_b_zp == 1 ? b_zp_host : b_zp_host + (size_t)g * Og, n_b_zp == 1 ? 1 : Og, Og, np,
                      go + (size_t)g * 2 * np + np, s, &unused);
      if (rc == QG_OK && qg_launch_pack_b(W_dev + (size_t)g * K * Og, K, Og, Og, 0, kp, np, gp + (size_t)g * kp * np,
                                          go + (size_t)g * 2 * np, go + (size_t)g * 2 * np + np, s) != hipSuccess)
        rc = QG_ELAUNCH;
      if (rc != QG_OK) {
        delete h;
        return rc;
      }
    }
    h->conv_gemm = gp;
    h->conv_gemm_off = go;
    h->conv_gemm_kpad = kp;
    h->conv_gemm_npad = np;
  }
  *out = h;
  return QG_OK;
}

int qg_conv_groupwise_u8s8_requant(const uint8_t* in_nhwc, int Nb, int H, int W, int C, int pad,
                                   int stride, const qg_packed_b* Wp, const qg_requant_params* p,
                                   uint8_t* out_nhwc, void* stream) {
  if (!Wp || ((!in_nhwc || !out_nhwc) && Nb != 0)) return QG_ENULL;
  if (Wp->kind != QG_KIND_CONV || Wp->version != QG_LAYOUT_VERSION) return QG_EINVAL;
  if (Nb < 0 || H <= 0 || W <= 0 || C <= 0 || pad < 0 || stride <= 0) return QG_EINVAL;
  if (C != Wp->G * Wp->Cg) return QG_EINVAL;
  int rc = check_requant(p, Wp->N);
  if (rc != QG_OK) return rc;
  const int Ho = (H + 2 * pad - Wp->R) / stride + 1;
  const int Wo = (W + 2 * pad - Wp->S) / stride + 1;
  if (H + 2 * pad < Wp->R || W + 2 * pad < Wp->S || Ho <= 0 || Wo <= 0) return QG_EINVAL;
  if (Wp->conv_any == nullptr && (!aligned(in_nhwc, 4) || !aligned(out_nhwc, 4))) return QG_EALIGN;
  if ((uint64_t)Nb * H * W * C >= (1ull << 31) || (uint64_t)Nb * Ho * Wo * Wp->N >= (1ull << 31)) return QG_EUNSUPPORTED;
  qg_conv_args a = {};
  a.in = in_nhwc;
  a.Wp = Wp->packed;
  a.Wfrag = Wp->conv_frags;
  a.col_off = Wp->col_off;
  a.bzp = Wp->bzp;
  a.bias = p->bias;
  a.scales = p->scales;
  a.out = out_nhwc;
  a.Nb = Nb;
  a.H = H;
  a.W = W;
  a.C = C;
  a.Ho = Ho;
  a.Wo = Wo;
  a.Cout = Wp->N;
  a.G = Wp->G;
  a.Wany = Wp->conv_any;
  a.Cg = Wp->Cg;
  a.Og = Wp->Og;
  a.R = Wp->R;
  a.S = Wp->S;
  a.lcg = Wp->conv_any == nullptr ? 2 : (Wp->conv_frags != nullptr ? conv_mfma_lcg(Wp->G, Wp->R, Wp->S, Wp->Cg, Wp->Og) : 0);
  a.pad = pad;
  a.stride = stride;
  a.scale_stride = p->n_scales == 1 ? 0 : 1;
  a.a_zp = p->a_zp;
  a.c_zp = p->c_zp;
  const int lo = p->relu ? p->c_zp : 0;
  a.clamp_lo = (float)(lo - p->c_zp);
  a.clamp_hi = (float)(255 - p->c_zp);
  a.has_bzp = Wp->has_bzp;
  if (Nb == 0) return QG_OK;  // an empty batch
  // wide groups: every group is a dense convolution of its own channel slice (16-byte chunks need aligned pixels)
  if (Wp->conv_gemm != nullptr && C % 16 == 0 && aligned(in_nhwc, 16) && (uint64_t)Nb * H * W * C < (1ull << 30) &&
      (uint64_t)Nb * Ho * Wo < (1ull << 31) / 4) {
    const size_t kp = (size_t)Wp->conv_gemm_kpad, np = (size_t)Wp->conv_gemm_npad;
    for (int g = 0; g < Wp->G; ++g) {
      const int32_t* off = Wp->conv_gemm_off + (size_t)g * 2 * np;
      rc = launch_conv_gemm(in_nhwc + (size_t)g * Wp->Cg, Nb * H * W * C - g * Wp->Cg, Nb, H, W, Wp->Cg, C, Wp->R, Wp->S, pad,
                            stride, Ho, Wo, Wp->conv_gemm + (size_t)g * kp * np, off, off + np, Wp->K, (int)kp, Wp->Og, (int)np,
                            Wp->has_bzp, p, g * Wp->Og, out_nhwc + (size_t)g * Wp->Og, Wp->N, QG_KERNEL_AUTO,
                            static_cast<hipStream_t>(stream));
      if (rc != QG_OK) return rc;
    }
    return QG_OK;
  }
  hipError_t e = qg_launch_conv_group(a, Wp->R * Wp->S, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? QG_OK : QG_ELAUNCH;
}

}  // extern "C"
