// Dense convolution over few input channels (the RGB image of a first layer, any channel count that is not a multiple
// of 16) with the im2col folded into LDS addressing.
//
// In NHWC the S * C bytes that one filter row of an output pixel covers are consecutive ("a run"), so the im2col row
// of a pixel is R runs, one per image row.  A workgroup stages the image rows its output tile touches in LDS once --
// shifted to int8, the padding of the real domain as theta_A bytes -- and the A operand of an MFMA is then 16
// consecutive bytes of such a staged row at (pixel base) + (run, piece): one LDS read from any byte address, no
// gather, no border test.  A run is cut into 16-byte pieces; the last piece of a run reads on past it, into whatever
// follows, and meets weights that are zero there: the packed (R*S*C) x Cout matrix, whose rows are contiguous in k, is
// re-cut once per workgroup into the same pieces (two 16-byte units of a column, funnel-shifted; zeros past the run).
// Piece u of the flattened (run, piece) list is the k half u & 1 of MFMA step u >> 1.
//
// What bounds it: at 8 x 224 x 224 x 3, 7 x 7, stride 2 -> 64 channels the bytes take 1.5 us and the MFMAs 0.7; the
// time is the chain of one workgroup, 448 of which are resident at once (cycles: addresses and requests 2000, their
// latency and the re-cut 2000, a block of 32 pixels 1400 + its output pipeline).  Measured, graph replay, theta_B = 0: 7.0 to
// 7.6 us, where the byte-gathering kernel, which spends about 27 vector instructions per byte of the im2col matrix, takes 21;
// one image 5.3 (9.3), 32 images 15 (65), 3 x 3 stride 2 -> 32 4.8 (9.6), 16 x 256 x 256 x 4, 7 x 7 stride 1 -> 64 28 (81).  With
// theta_B, whose row sums are one more MFMA per step and leave the steps to a loop: 8.6 (22), 32 images 18 (69), 3 x 3 5.4
// (10.2), the last 36 (86).
#include "qg_internal.h"
#include <cmath>
#include <type_traits>

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

struct runs_args {
  const int32_t* col_off;
  const int32_t* bzp;
  const int32_t* bias;
  const float* scales;
  uint8_t* out;
  int Ho, Wo, Cout, steps;  // steps: MFMA steps of two pieces
  int scale_stride, c_zp;
  float clamp_lo, clamp_hi, inv_tw;
};

// byte mask of a dword: its first n bytes (n <= 0: none, n >= 4: all)
__device__ __forceinline__ unsigned first_bytes(int n) { return n >= 4 ? 0xFFFFFFFFu : (n <= 0 ? 0u : (1u << (8 * n)) - 1u); }

// 16 consecutive LDS bytes from p + sh, p a multiple of 4 and sh in 0..3: whole dwords and a funnel shift.  (A 16-byte
// LDS read from an odd address works but costs the LDS about 70 cycles, where the five dwords of this one cost 10.)
__device__ __forceinline__ v4i lds_bytes16(const unsigned char* p, unsigned sh) {
  const unsigned* w = reinterpret_cast<const unsigned*>(p);
  const unsigned d0 = w[0], d1 = w[1], d2 = w[2], d3 = w[3], d4 = w[4];
  return (v4i){(int)__builtin_amdgcn_alignbyte(d1, d0, sh), (int)__builtin_amdgcn_alignbyte(d2, d1, sh),
               (int)__builtin_amdgcn_alignbyte(d3, d2, sh), (int)__builtin_amdgcn_alignbyte(d4, d3, sh)};
}

// KS: MFMA steps, the weight operands then stay in registers over all pixel blocks of a wave (0: any number, from LDS).
// NB: blocks of 32 output channels per workgroup.
template <int KS, int NB, bool HAS_BZP, int NT, bool HOLD>
__global__ __launch_bounds__(NT, NT == 256 ? (HOLD ? 2 : 4) : 2) void qg_conv_runs_kernel(
    const uint8_t* in, const int8_t* Bp, const int H, const int rowlen, const int pxstep, const int stride_pad, const int b_first,
    const int pitch, const float inv_cpr, const int TW_TH, const int nx_R, const int in_bytes, const int run_m, const int nb16,
    const int azp, const runs_args p) {
  // the leading scalar arguments hold what the loads below need: the file is compiled with kernel-argument preloading, so
  // they arrive in scalar registers with the wave
  extern __shared__ __align__(16) unsigned char smem[];
  const int steps = KS > 0 ? KS : p.steps;
  unsigned char* const w_s = smem;                                       // [piece][64 slots] x 16 bytes
  int* const cj_s = reinterpret_cast<int*>(smem + steps * 2048);
  int* const nbz_s = cj_s + 64;
  float* const sc_s = reinterpret_cast<float*>(nbz_s + 64);
  v4i* const ones_s = reinterpret_cast<v4i*>(sc_s + 64);                 // HAS_BZP: [piece], 1 at the bytes of the run
  unsigned char* const patch = smem + steps * 2048 + 768 + (HAS_BZP ? steps * 32 : 0);
  constexpr int NWAVE = NT / 64;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lg = lane >> 5;
  const int TW = TW_TH & 0xFFFF, TH = TW_TH >> 16, nx = nx_R & 0xFFFF, R = nx_R >> 16;
  const int stride = stride_pad & 0xFFFF, pad = (int)((unsigned)stride_pad >> 16), run = run_m & 0xFFFF;
  const int up = (run + 15) >> 4;          // pieces of a run
  const int nblk = nx > 1 ? (int)blockIdx.x / nx : (int)blockIdx.x, tx = (int)blockIdx.x - nblk * nx;
  const int n0 = nblk * (NB * 32), n = blockIdx.z;
  const int ho0 = blockIdx.y * TH, wo0 = tx * TW;
  const int h0 = ho0 * stride - pad;       // image row of patch row 0
  const int b0 = wo0 * pxstep + b_first;   // position in an image row of a patch row's first byte (may be negative)
  const int prows = (TH - 1) * stride + R, cpr = pitch >> 4, nchunks = prows * cpr;
  const int row0 = n * H + h0;

  // ---- the patch: 16-byte chunks from any address, shifted to int8, what lies outside the image as theta_A.  A chunk at
  // the edge of an image row is loaded whole, neighbouring bytes included, and those masked out behind the load -- unless
  // that would leave the buffer: then only its bytes inside are read, one by one.
  struct chunk {
    v4i v;
    int pos;  // position of its first byte in the image row; rowlen when nothing of it is inside
  };
  auto load_chunk = [&](int c) {
    chunk k;
    const int r = (int)(((float)c + 0.5f) * inv_cpr), cc = c - r * cpr;
    k.pos = b0 + cc * 16;
    const int off = (row0 + r) * rowlen + k.pos;
    k.v = (v4i){0, 0, 0, 0};
    if ((unsigned)(h0 + r) >= (unsigned)H || c >= nchunks) k.pos = rowlen;
    if (k.pos < rowlen) {
      if (off >= 0 && off <= in_bytes - 16) {
        k.v = *reinterpret_cast<const qg_v4i_unaligned*>(in + off);
      } else {
        for (int i = 0; i < 16; ++i)
          if (k.pos + i >= 0 && k.pos + i < rowlen) k.v[i >> 2] |= (int)((unsigned)in[off + i] << (8 * (i & 3)));
      }
    }
    return k;
  };
  auto store_chunk = [&](int c, chunk k) {
    if (c >= nchunks) return;
    if (k.pos < 0 || k.pos + 16 > rowlen) {
      const unsigned azp4 = (unsigned)azp * 0x01010101u;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const unsigned keep = first_bytes(rowlen - k.pos - 4 * d) & ~first_bytes(-k.pos - 4 * d);
        k.v[d] = (int)(((unsigned)k.v[d] & keep) | (azp4 & ~keep));
      }
    }
    *reinterpret_cast<v4i*>(patch + c * 16) = k.v ^ (int)0x80808080;
  };
  const chunk c0 = load_chunk(tid), c1 = load_chunk(tid + NT);

  // ---- the weights, re-cut into pieces: lane = slot of one of the 64 columns, one piece per wave and pass.  Piece `lane`
  // (there are at most 48): its run, first k, number of bytes of the run from there on, and place in the patch
  const int p_kh = (lane * (int)((unsigned)run_m >> 16)) >> 15, p_in = (lane - p_kh * up) * 16;
  const int p_k0 = p_kh * run + p_in, p_nv = p_kh < R ? run - p_in : 0, p_off = p_kh < R ? p_kh * pitch + p_in : 0;
  const int8_t* const wbase = Bp + (size_t)(n0 >> 4) * QG_FRAG_BYTES;
  const int wlane = (lane >> 4) * QG_FRAG_BYTES + (lane & 15) * 16;
  const size_t slab = (size_t)nb16 * QG_FRAG_BYTES;
  struct piece {
    v4i lo, hi;
    int k0, nv;
  };
  auto load_piece = [&](int u) {  // the one or two 16-byte units of a packed column that the piece reaches into
    piece w;
    w.k0 = __builtin_amdgcn_readlane(p_k0, u);
    w.nv = __builtin_amdgcn_readlane(p_nv, u);
    if (w.nv > 0) {
      const int ku = w.k0 >> 4;
      const int8_t* const src = wbase + (size_t)(ku >> 2) * slab + (ku & 3) * 256;
      w.lo = *reinterpret_cast<const v4i*>(src + wlane);
      // (behind the last unit there is nothing: where the piece ends in the first one, that one again)
      const size_t next = (w.k0 & 15) + min(w.nv, 16) <= 16 ? (size_t)0 : ((ku & 3) == 3 ? slab - 768 : (size_t)256);
      w.hi = *reinterpret_cast<const v4i*>(src + next + wlane);
    }
    return w;
  };
  auto store_piece = [&](int u, const piece& w) {
    v4i o = (v4i){0, 0, 0, 0};
    if (w.nv > 0) {
      unsigned d[8] = {(unsigned)w.lo.x, (unsigned)w.lo.y, (unsigned)w.lo.z, (unsigned)w.lo.w,
                       (unsigned)w.hi.x, (unsigned)w.hi.y, (unsigned)w.hi.z, (unsigned)w.hi.w};
      if (w.k0 & 8) {
#pragma unroll
        for (int i = 0; i < 6; ++i) d[i] = d[i + 2];
      }
      if (w.k0 & 4) {
#pragma unroll
        for (int i = 0; i < 5; ++i) d[i] = d[i + 1];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = (int)__builtin_amdgcn_alignbyte(d[i + 1], d[i], w.k0 & 3);
      if (w.nv < 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = (int)((unsigned)o[i] & first_bytes(w.nv - 4 * i));
      }
    }
    *reinterpret_cast<v4i*>(w_s + u * 1024 + lane * 16) = o;
    if (HAS_BZP && lane == 0)
      ones_s[u] = (v4i){(int)(first_bytes(w.nv) & 0x01010101u), (int)(first_bytes(w.nv - 4) & 0x01010101u),
                        (int)(first_bytes(w.nv - 8) & 0x01010101u), (int)(first_bytes(w.nv - 12) & 0x01010101u)};
  };
  constexpr int WP = KS > 0 ? (2 * KS + NWAVE - 1) / NWAVE : 1;  // pieces per wave: their loads are issued here, behind the patch's
  piece w[WP];
#pragma unroll
  for (int i = 0; i < WP; ++i) w[i] = load_piece(wave + NWAVE * i);  // (one too many: lane u has nv = 0)
  int cj = 0, nbz = 0;
  float sc = 0.0f;
  const int col = n0 + tid;
  if (tid < NB * 32 && col < p.Cout) {
    cj = (p.bias ? p.bias[col] : 0) - (azp - 128) * p.col_off[col];
    if (HAS_BZP) nbz = -p.bzp[col];
    sc = p.scales[(size_t)col * p.scale_stride];
  }

  store_chunk(tid, c0);
  store_chunk(tid + NT, c1);
  for (int c = tid + 2 * NT; c < nchunks; c += 2 * NT) {
    const chunk ca = load_chunk(c), cb = load_chunk(c + NT);
    store_chunk(c, ca);
    store_chunk(c + NT, cb);
  }
#pragma unroll
  for (int i = 0; i < WP; ++i)
    if (wave + NWAVE * i < 2 * steps) store_piece(wave + NWAVE * i, w[i]);
  if constexpr (KS == 0) {
    for (int u = wave + NWAVE; u < 2 * steps; u += NWAVE) store_piece(u, load_piece(u));
  }
  if (tid < NB * 32) {
    cj_s[tid] = cj;
    if (HAS_BZP) nbz_s[tid] = nbz;
    sc_s[tid] = sc;
  }
  const int th = min(TH, p.Ho - ho0), tw = min(TW, p.Wo - wo0), npx = th * TW;
  const float inv_tw = p.inv_tw, czp_f = (float)p.c_zp;
  const bool vec_out = (((uintptr_t)p.out | (uintptr_t)p.Cout) & 15) == 0;
  uint8_t* const out0 = p.out + ((size_t)n * p.Ho + ho0) * p.Wo * p.Cout + (size_t)wo0 * p.Cout;
  __syncthreads();

  v4i wf[KS > 0 && HOLD ? KS : 1][NB];
  int aoff[KS > 0 ? KS : 1];
  if constexpr (KS > 0) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      aoff[ks] = lg ? __builtin_amdgcn_readlane(p_off, 2 * ks + 1) : __builtin_amdgcn_readlane(p_off, 2 * ks);
#pragma unroll
      for (int nb = 0; HOLD && nb < NB; ++nb)
        wf[ks][nb] = *reinterpret_cast<const v4i*>(w_s + (2 * ks + lg) * 1024 + (nb * 32 + l32) * 16);
    }
  }

  for (int blk = wave; blk * 32 < npx; blk += NWAVE) {
    const int t = min(blk * 32 + l32, npx - 1);
    const int hl = (int)(((float)t + 0.5f) * inv_tw), wl = t - hl * TW;
    const int ab = hl * stride * pitch + wl * pxstep;
    const unsigned char* const a0 = patch + (ab & ~3);
    const unsigned sh = (unsigned)ab & 3u;  // pitch and pieces are multiples of 16: the same for every piece
    v16i acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const v4i cjv = *reinterpret_cast<const v4i*>(&cj_s[nb * 32 + 16 * lg + 4 * q]);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[nb][4 * q + r] = cjv[r];
      }
    v16i racc;
    if (HAS_BZP) {
#pragma unroll
      for (int r = 0; r < 16; ++r) racc[r] = 0;
    }
    auto wfrag = [&](int ks, int nb) { return *reinterpret_cast<const v4i*>(w_s + (2 * ks + lg) * 1024 + (nb * 32 + l32) * 16); };
    if constexpr (KS > 0) {
      v4i a[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) a[ks] = lds_bytes16(a0 + aoff[ks], sh);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(HOLD ? wf[HOLD ? ks : 0][nb] : wfrag(ks, nb), a[ks], acc[nb], 0, 0, 0);
      }
    } else {
      for (int ks = 0; ks < steps; ++ks) {
        const int o0 = __builtin_amdgcn_readlane(p_off, 2 * ks), o1 = __builtin_amdgcn_readlane(p_off, 2 * ks + 1);
        const v4i a = lds_bytes16(a0 + (lg ? o1 : o0), sh);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wfrag(ks, nb), a, acc[nb], 0, 0, 0);
        if (HAS_BZP) racc = __builtin_amdgcn_mfma_i32_32x32x32_i8(ones_s[2 * ks + lg], a, racc, 0, 0, 0);
      }
    }
    // lane (pixel l32, half lg) holds 16 consecutive output channels of its pixel; every register of racc holds the
    // byte sum of the pixel's row in the int8 domain
    if (blk * 32 + l32 < npx && wl < tw) {
      uint8_t* const dst0 = out0 + ((size_t)hl * p.Wo + wl) * p.Cout;
      auto pipeline = [&](auto form_tag) {
        constexpr int FORM = decltype(form_tag)::value;  // 0: explicit clamp, 1: saturating convert, 2: theta_C == 0
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int c_l = nb * 32 + lg * 16, col0 = n0 + c_l;
          unsigned o[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float4 sc = *reinterpret_cast<const float4*>(&sc_s[c_l + 4 * q]);
            const float s4[4] = {sc.x, sc.y, sc.z, sc.w};
            unsigned w = 0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              int x = acc[nb][4 * q + r];
              if (HAS_BZP) x += nbz_s[c_l + 4 * q + r] * racc[0];
              if (FORM == 2)
                w = qg_requant_pack0(x, s4[r], r, w);
              else
                w = qg_requant_pack<FORM == 0>(x, s4[r], p.clamp_lo, p.clamp_hi, czp_f, r, w);
            }
            o[q] = w;
          }
          uint8_t* const dst = dst0 + col0;
          if (vec_out && col0 + 16 <= p.Cout) {
            *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
          } else {
#pragma unroll
            for (int i = 0; i < 16; ++i)
              if (col0 + i < p.Cout) dst[i] = (uint8_t)(o[i >> 2] >> (8 * (i & 3)));
          }
        }
      };
      if (qg_requant_needs_lo(p.clamp_lo, czp_f))
        pipeline(std::integral_constant<int, 0>{});
      else if (p.c_zp == 0)
        pipeline(std::integral_constant<int, 2>{});
      else
        pipeline(std::integral_constant<int, 1>{});
    }
  }
}

struct runs_plan {
  runs_args p;
  int rowlen, pxstep, pitch, run, TW, TH, nx, ny, nb, smem;
  bool full;
};

// Tile and LDS of a layer; false when the weights or the patch do not fit.
bool plan_runs(const qg_conv_args& a, runs_plan* pl) {
  runs_args& p = pl->p;
  pl->run = a.S * a.C;
  const int up = (pl->run + 15) / 16;
  p.steps = (a.R * up + 1) / 2;
  if (p.steps > 24 || a.R > 0x7FFF || a.stride > 0x7FFF || a.pad > 0x7FFF) return false;
  pl->nb = a.Cout > 32 ? 2 : 1;
  pl->rowlen = a.W * a.C;
  pl->pxstep = a.stride * a.C;
  const long long npix = (long long)a.Nb * a.Ho * a.Wo;
  // output pixels per workgroup, 64 to 512: two workgroups per CU, one where re-cutting the weights is most of the set-up
  // (8 x 56 x 56 x 24, 3 x 3 -> 24, 8 steps, run on this kernel: 5.1 us against 5.6; 8 x 224 x 224 x 4, 7 x 7, stride 2 -> 64, 7 steps: 7.3
  // against 6.7)
  const long long ncol = (a.Cout + pl->nb * 32 - 1) / (pl->nb * 32);
  long long target = npix * ncol / (p.steps >= 8 ? 256 : 512);
  if (target < 64) target = 64;
  if (target > 512) target = 512;
  pl->full = target == 512;
  for (;; target /= 2) {
    if (target < 32) return false;
    if (a.Wo <= target) {
      pl->nx = 1;
      pl->TW = a.Wo;
      pl->TH = (int)((target + a.Wo / 2) / a.Wo);
      if (pl->TH > a.Ho) pl->TH = a.Ho;
    } else {
      pl->TW = (int)((a.Wo + (a.Wo + target - 1) / target - 1) / ((a.Wo + target - 1) / target));
      pl->nx = (a.Wo + pl->TW - 1) / pl->TW;
      pl->TH = 1;
    }
    pl->ny = (a.Ho + pl->TH - 1) / pl->TH;
    const long long pitch = ((long long)(pl->TW - 1) * pl->pxstep + pl->run + 15) / 16 * 16;
    const long long prows = (long long)(pl->TH - 1) * a.stride + a.R;
    const long long smem = p.steps * 2048 + 768 + (a.has_bzp ? p.steps * 32 : 0) + pitch * prows + 32;
    if (smem > 80 * 1024) continue;  // two workgroups per CU
    pl->pitch = (int)pitch;
    pl->smem = (int)smem;
    break;
  }
  if (a.Nb > 65535 || pl->ny > 65535 || pl->nx > 0xFFFF) return false;
  p.col_off = a.col_off;
  p.bzp = a.bzp;
  p.bias = a.bias;
  p.scales = a.scales;
  p.out = a.out;
  p.Ho = a.Ho;
  p.Wo = a.Wo;
  p.Cout = a.Cout;
  p.scale_stride = a.scale_stride;
  p.inv_tw = 1.0f / (float)pl->TW;
  p.c_zp = a.c_zp;
  p.clamp_lo = a.clamp_lo;
  p.clamp_hi = a.clamp_hi;
  return true;
}

template <int KS, int NB, bool HAS_BZP, int NT, bool HOLD>
hipError_t launch_runs(const qg_conv_args& a, const runs_plan& pl, hipStream_t s) {
  constexpr auto fn = qg_conv_runs_kernel<KS, NB, HAS_BZP, NT, HOLD>;
  if (hipError_t e = qg_allow_smem<fn>(pl.smem); e != hipSuccess) return e;
  const dim3 grid((unsigned)(pl.nx * ((a.Cout + NB * 32 - 1) / (NB * 32))), (unsigned)pl.ny, (unsigned)a.Nb);
  const int up = (pl.run + 15) / 16, m = (32768 + up - 1) / up;  // u / up == u * m >> 15 for the at most 48 pieces u
  hipLaunchKernelGGL(fn, grid, dim3(NT), pl.smem, s, a.in, a.Bp, a.H, pl.rowlen, pl.pxstep, a.stride | (a.pad << 16), -a.pad * a.C,
                     pl.pitch, 16.0f / (float)pl.pitch, pl.TW | (pl.TH << 16), pl.nx | (a.R << 16), a.Nb * a.H * a.W * a.C,
                     pl.run | (m << 16), a.nb16, a.a_zp, pl.p);
  return hipGetLastError();
}
// Eight waves per workgroup, the weight operands read from LDS for every block; few steps over very many pixels take four
// waves that hold them in registers (8 x 224 x 224 x 3, 3 x 3, stride 1 -> 32: 7.3 us against 7.9; at 7 steps, 8 x 224 x
// 224 x 3, 7 x 7, stride 2 -> 64, the eight waves win: 7.0 against 7.5).
template <int KS, int NB>
hipError_t launch_runs_few(const qg_conv_args& a, const runs_plan& pl, hipStream_t s) {
  return pl.full ? launch_runs<KS, NB, false, 256, true>(a, pl, s) : launch_runs<KS, NB, false, 512, false>(a, pl, s);
}
template <int NB>
hipError_t launch_runs_ks(const qg_conv_args& a, const runs_plan& pl, hipStream_t s) {
  if (a.has_bzp) return launch_runs<0, NB, true, 512, false>(a, pl, s);
  switch (pl.p.steps) {
    case 1: return launch_runs_few<1, NB>(a, pl, s);
    case 2: return launch_runs_few<2, NB>(a, pl, s);
    case 3: return launch_runs_few<3, NB>(a, pl, s);
    case 4: return launch_runs<4, NB, false, 512, false>(a, pl, s);
    case 5: return launch_runs<5, NB, false, 512, false>(a, pl, s);
    case 7: return launch_runs<7, NB, false, 512, false>(a, pl, s);
    case 8: return launch_runs<8, NB, false, 512, false>(a, pl, s);
    default: return launch_runs<0, NB, false, 512, false>(a, pl, s);  // (6 and 9 .. 24: few layers have them)
  }
}

}  // namespace

// Microseconds of this kernel on a planned layer, and of the byte-gathering kernel on the same one (without the time of the
// stores, which is the same for both): launch, then the larger of a workgroup's own chain and what the workgroups of a CU share.
// Constants fitted to 3270 drawn layers, C 1 .. 72, filters 2 x 1 .. 16 x 17, strides 1 .. 16, with and without theta_B.
namespace {
double runs_estimate(const qg_conv_args& a, const runs_plan& pl) {
  const int steps = pl.p.steps, px = pl.TW * pl.TH;
  const bool held = pl.full && steps <= 3 && !a.has_bzp, any_steps = a.has_bzp || steps > 8 || steps == 6;
  const int waves = held ? 4 : 8, chunks = pl.pitch / 16 * ((pl.TH - 1) * a.stride + a.R);
  const double mfma = steps * pl.nb * (a.has_bzp ? 1.92 : 1.0);
  const double chain = 0.325 * ((chunks + waves * 128 - 1) / (waves * 128)) + (any_steps ? 0.075 : 0.038) * steps +
                       0.0355 * mfma * (((px + 31) / 32 + waves - 1) / waves);
  const double share = 0.195 + 0.244 * chunks / 512 + 0.096 * steps + ((px + 31) / 32) / 8.0 * (0.505 + 0.06 * mfma);
  const int by_lds = 160 * 1024 / pl.smem, by_waves = held ? 5 : 3, per_cu = by_lds < by_waves ? by_lds : by_waves;
  const double wgs = (double)pl.nx * pl.ny * a.Nb * ((a.Cout + pl.nb * 32 - 1) / (pl.nb * 32)) / 256.0;  // per CU
  const double rounds = floor(wgs / per_cu), left = fmin(wgs - rounds * per_cu, (double)per_cu);
  return 3.95 + rounds * fmax(chain, per_cu * share) + (left > 0.0 ? fmax(chain, left * share) : 0.0);
}
double gather_estimate(const qg_conv_args& a) {
  const bool words = a.C % 4 == 0 && ((uintptr_t)a.in & 3) == 0;
  const double kt = (a.R * a.S * a.C + 63) / 64, wgs = (double)(((long long)a.Nb * a.Ho * a.Wo + 63) / 64) * ((a.Cout + 63) / 64) / 256.0;
  return words ? 2.7 + fmax(kt * (a.has_bzp ? 0.75 : 0.64), wgs * (kt * 0.29 + 0.38))
               : 2.9 + fmax(kt * (a.has_bzp ? 2.41 : 2.06), wgs * (kt * 0.79 + 0.39));
}
}  // namespace

// Not for 1 x 1 filters (nothing overlaps: 4 x 28 x 28 x 40, stride 2 -> 72 takes 4.0 us here, 3.7 on the gathering
// kernel), nor where the weights of one column block outgrow the LDS (more than 48 pieces); otherwise where the estimate is
// 5 % ahead.  Gathering stays ahead where it loads whole words over a short K and the set-up here is not shared by many
// pixels (3 x 219 x 219 x 4, 5 x 5, stride 2 -> 16 4.8 us against 7.5 here), and for strides beyond the filter, whose rows
// hold much that is not needed (250 x 32 x 72 x 24, 2 x 2, stride 8 -> 192 5.3 against 14.4).  Over the drawn layers 0.72 of the
// gathering kernel's time in the mean, 1 % behind the better of the two.
// Columns that end inside a 16-byte store are written byte by byte; where that bounds both kernels, the column blocks of a
// pixel, side by side here, write into the same lines from different XCDs (32 x 94 x 91 x 12, 2 x 2 -> 72 66.5 us, 101 here).
bool qg_conv_runs_applies(const qg_conv_args& a) {
  runs_plan pl;
  if (a.R * a.S == 1 || !plan_runs(a, &pl)) return false;
  const double gather_us = gather_estimate(a);
  const bool byte_stores = a.Cout % 16 != 0 || ((uintptr_t)a.out & 15) != 0;
  if (byte_stores && a.Cout > 64 && (double)a.Nb * a.Ho * a.Wo * a.Cout * 3.9e-6 > gather_us) return false;
  return runs_estimate(a, pl) * 1.05 < gather_us;
}

hipError_t qg_launch_conv_runs(const qg_conv_args& a, hipStream_t s) {
  runs_plan pl;
  if (!plan_runs(a, &pl)) return hipErrorInvalidValue;
  return pl.nb == 2 ? launch_runs_ks<2>(a, pl, s) : launch_runs_ks<1>(a, pl, s);
}
