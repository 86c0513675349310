// Small-batch quantized GEMM (row blocks of 16, 32 or 64): the bandwidth-bound case the paper
// stresses ("M is sometimes very small", Appendix C; int32 accumulation for the
// bandwidth-bound shapes, Sec. 4).  Every byte of B is used exactly once, so B
// fragments go STRAIGHT from HBM into MFMA operand registers: the packed layout
// makes each wave load one contiguous KiB (16 B per lane).
//
// One workgroup owns one or two 16-column fragment columns of B over all of K; its 4 to 16 waves split K, and wave w
// takes a contiguous range of 64-deep k blocks and issues a whole batch of loads
// before the first MFMA so that the whole weight matrix is in flight at once; the next
// batch is requested before the wave waits for the current one.
// A (the row block, at most 64 rows) comes from L2, is row-summed on its raw bytes (v_sad_u8) and
// shifted to int8 (xor 0x80) on the way, as in the large kernel.  Each wave stages its own K-slice of
// the row block, batch by batch, through a private 4 or 8 KiB of LDS with global_load_lds: a request
// reads whole 128- or 256-byte row segments (MFMA operand order would touch 16 rows x 64 B per load,
// half-used lines, which cost more than the weight stream itself at 64 rows), and the fragments are then
// fetched from LDS in operand order.  Rows at any address, any K and batches that K cuts take the same route (SRC_U8 below): copied
// by the lanes, chunk by chunk and at the end of K byte by byte, such a batch held up its whole workgroup (1 x 4320 x 4122
// 9.7 -> 5.8 us, 42 x 1408 x 5897 14.0 -> 7.4).
//
// Outlier-split weights (Sec. 2.2, B = B' + B_sparse): B' streams in at 4 bits per weight -- half the bytes
// of the shape this kernel exists for -- and is widened to int8 operand dwords with two bit operations
// per eight weights; the sparse term A B_sparse is added while the block of C is still on chip (the paper
// fuses it into the output processing while the block is cache-resident): a wave that has just consumed a
// batch of k blocks scatters that batch's entries, one per lane and byte store, into zeroed fragments in its staging
// region (the activations are in registers by then) and multiplies those like any other weights.  One product per
// (row, entry) pair and lane, added up in LDS, was what this took before: vector instructions, 16 rows of them per
// entry, bound it (16 x 8192 x 8192, weights in the memory-side cache, with 0.7 % of outliers 17.5 -> 10.9 us; 0.1 % 10.8, 1 %
// 11.2, 2 %, more than 64 entries in some batches, 13.2, and none at all, where batches skip this, 8.5; with 0.5 % 64 x 4096 x 4096
// 13.4 -> 7.7, 64 x 8192 x 8192 44 -> 20).  What is left is the chain request, widen, scatter, read of a batch; with the next batch's
// requests in flight meanwhile and two columns per wave 16 x 8192 x 8192 with 0.5 % takes 10.3 us (13.3 before), 64 x 4864 x 6912 14.2 (17.6).
//
// M larger than the row block is covered by the second grid dimension: every row block streams
// B again (from L2 / the memory-side cache when the blocks run close together), which beats the
// tiled kernel only while there are too few tiles to occupy the chip.
//
// K split ACROSS workgroups (third grid dimension, p.ksplit slices of K; the role of the paper's caller-provided
// C_buffer, Appendix A): a shape with few fragment columns and a long K would leave most of the chip idle, so the
// slices of one fragment column run as separate workgroups.  Each adds up its own waves through LDS as usual; the
// wave that would run the output pipeline instead writes its int32 partial tile and row offsets into its slot of
// the caller's workspace with device-coherent (write-through) stores, waits for their acknowledgement and takes
// a ticket from a counter; the wave that draws the last ticket reads the other slices' slots, adds them in slice
// order -- integer sums, so every split factor gives the same bytes -- runs the output pipeline and puts the
// counter back to zero for the next call.  No fence instruction is used: a release fence at device scope writes
// back the whole L2 of the XCD, which was measured at 20 - 80 us per workgroup.
#include "qg_internal.h"
#include <type_traits>

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

// ints of one (K slice, row block of 16) slot of the cross-workgroup workspace: 64 lanes x 4 partial sums, 16 row sums
constexpr int SLOT_INTS = 64 * 4 + 16;

// One activation request: 16 bytes per lane from a_base + voff (a_base wave-uniform, in scalar registers; voff a
// per-lane byte offset) into LDS at lds + lane * 16 (lds wave-uniform).  Written out instead of the compiler's
// builtin because that one forms the 64-bit address in a temporary vector register, and the register it picked
// was the destination of a weight load still in flight: the request then waited for weights from HBM before it
// could even be issued.  Here the address registers are never the target of a load.
__device__ __forceinline__ void request_a(const uint8_t* a_base, unsigned voff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(voff), "s"(a_base) : "memory");
}

// The same with a 64-bit per-lane address (requests that may go to a table row).
__device__ __forceinline__ void request_a64(const uint8_t* addr, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(addr) : "memory");
}

// 4 bytes per lane, to lds + lane * 4
__device__ __forceinline__ void request_dword(const void* addr, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds), "v"(addr) : "memory");
}

// Explicit wait: at most LEFT vector-memory operations of this wave still in flight (they complete in order).
// The compiler's own bookkeeping does not see the activation requests (they are issued by request_a), so the
// waits that order LDS reads behind them are written out.
template <int LEFT>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LEFT) : "memory");
}

// SRC: what a row of the staged block is.
// SRC_U8: a row of A, from any address.  A batch that reaches past K requests the chunks behind it from a row of 0x80 bytes (the
// int8 zero after the shift); the chunk that K cuts is loaded once, at the start, as the last 16 bytes of its row, and put in place
// when its batch has arrived.
// SRC_F32: fp32 activations, quantized to uint8 while they are staged (Appendix B: any packing routine for A; Eq. (1) solved for
// the quantized value, the fixed sequence of the stand-alone quantization pass).  A then points to floats and lda counts
// floats; a lane loads four consecutive floats, so that a load of the wave is 1 KiB of a row, and writes one dword of LDS.
// SRC_CONV: the rows are the output pixels of a dense convolution and A is its NHWC image (the paper names convolution in
// Sec. 1; im2col folded into the requests as in the tiled kernels): the K = R*S*Cin bytes of a row are R*S runs of
// Cin channels (Cin a multiple of 64, so every 64-deep k block lies inside one filter tap), and the 16-byte chunk a
// lane requests comes from its pixel at that tap, or from a constant row of theta_A bytes when the tap lies outside
// the image (a k block past K: of 0x80 bytes, the K padding).  A request here covers ONE k block for 16 rows (lane =
// row, 16-byte piece of the block), so the tap of a request is wave-uniform and lives on the scalar unit, moved on
// block by block; a lane carries its pixel's byte offset and one validity bit per tap (R*S <= 32) per row block.
// The staged batch is therefore laid out [k block][row block][16 rows][64 bytes] instead of whole row segments.
// CPW: fragment columns per wave.  With two, a workgroup covers a whole 32-column super-block: every activation fragment feeds
// two MFMAs, the workgroup stages half as many activation bytes per weight byte, and few fat waves (16 weight loads in flight
// each) keep a large matrix streaming at the rate of a plain read -- the shape for more workgroups than CUs.
// DB: two staging regions per wave, so that a batch's activations are requested one batch ahead like its weights.
// WHOLE: every wave of every slice has whole batches and nothing that K could cut (checked by the host): any number with DB or with
// batches of eight, otherwise one, straight code then.
// SRC_CONV16: the same for any multiple of 16 channels.  A k block may then hold pieces of several taps, so the tap is per-lane
// state, moved on by four 16-byte pieces per block (2 x 12 x 12 x 96 -> 128, 3 x 3, stride 2: 6.3 us on the tiles, 4.2 here).
constexpr int SRC_U8 = 0, SRC_F32 = 1, SRC_CONV = 2, SRC_CONV16 = 3;
template <int MODE, int MB, int NWAVES, int BATCH, int CPW, bool B4, int SRC, bool DB, bool WHOLE = false>
__global__ __launch_bounds__(NWAVES * 64, NWAVES == 4 ? (MB == 1 ? 2 : 1) : NWAVES / 4) void qg_gemm_skinny_kernel(
    const uint8_t* A, const int8_t* Bp, const int M, const int N, const int K, const int kb64, const int nb16_total, const int lda,
    const int ks_per, const int ksplit, const qg_gemm_args p) {
  // The leading scalar arguments repeat what a wave needs before it can issue its first loads (the fields of the same
  // names in p): the file is compiled with kernel-argument preloading, so they arrive in scalar registers with the
  // wave instead of costing a cold trip to memory (measured: 0.4 us of a 5 us launch).
  static_assert(!B4 || (SRC == SRC_U8 && DB), "4-bit weights: rows of bytes, all requests of a batch one batch ahead");
  static_assert(!WHOLE || (SRC == SRC_U8 && !B4), "whole batches of 8-bit weights and rows of bytes");
  static_assert(SRC != SRC_F32 || !DB, "fp32 rows pass through registers, batch by batch");
  static_assert(MB * CPW <= NWAVES, "one wave per (row block, fragment column) runs the output pipeline");
  constexpr bool CONV = SRC == SRC_CONV || SRC == SRC_CONV16, ONE = WHOLE && !DB && BATCH < 8;
  // A through LDS (see the file header): per wave and batch, ROWS rows x ROWB bytes
  constexpr int ROWS = MB * 16, ROWB = BATCH * QG_FRAG_K, NCHUNK = ROWB / 16;
  constexpr int REGION = ROWS * ROWB, NREQ = REGION / 1024, RPR = 64 / NCHUNK;  // requests per batch, rows per request
  static_assert(NCHUNK == 8 || NCHUNK == 16 || NCHUNK == 32, "a request covers whole rows of 128, 256 or 512 bytes");
  constexpr int WAVE_LDS = REGION * (DB ? 2 : 1);
  // every wave leaves its K-split partial sums (MB * CPW KiB) at the start of its OWN staging region once
  // it is done with it: no wave waits for the others before it may write
  static_assert(MB * CPW * 1024 <= WAVE_LDS, "a wave's partial tile fits its staging region");
  static_assert(!B4 || REGION >= BATCH * QG_FRAG_BYTES, "the scattered fragments of a batch and column fit the wave's region");
  extern __shared__ __align__(16) unsigned char smem[];
  int* rsp = reinterpret_cast<int*>(smem + NWAVES * WAVE_LDS);    // [mb][row][wave]

  const int nb16 = blockIdx.x * CPW;  // first fragment column of this workgroup
  // columns held by fragment f: (f>>1)*32 + 16*(u&1) + 8*(f&1) + 4*(u>>1) + r, u<4, r<4
  if ((nb16 >> 1) * 32 + 8 * (nb16 & 1) >= N) return;  // nothing but padding (uniform for the workgroup)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ml = lane & 15, g = lane >> 4;
  const int m_base = blockIdx.y * (MB * 16);  // first row of this workgroup's row block

  // The waves that run the output pipeline request its per-column constants early, not after the reduction -- but
  // BEHIND the first batch's weight loads and activation requests: cold, they take a trip to HBM.  One request straight to LDS, 16
  // columns of the four arrays, so that nothing waits for them and no registers are held (16 loads per lane before).
  // wave w < MB * CPW runs the output pipeline of row block w / CPW, fragment column nb16 + w % CPW
  const int red_mb = wave / CPW, red_c = wave % CPW;
  const int c0 = ((nb16 + red_c) >> 1) * 32 + 16 * (g & 1) + 8 * ((nb16 + red_c) & 1) + 4 * (g >> 1);  // this lane's 4 output columns
  int* const ep_s = rsp + NWAVES * ROWS + wave * 64;  // [column offset, theta_B, bias, scale][16 columns], waves w < MB * CPW
  auto request_ep = [&]() {
    if (wave < MB * CPW) {
      const int u = (lane >> 2) & 3, col = ((nb16 + red_c) >> 1) * 32 + 16 * (u & 1) + 8 * ((nb16 + red_c) & 1) + 4 * (u >> 1) + (lane & 3);
      // col_off / bzp are padded to N_pad, bias / scales are not
      const void* src = (g == 0 ? p.col_off : p.bzp) + col;
      if (MODE != QG_MODE_ACC32) {
        if (g == 2) src = p.bias != nullptr && col < N ? static_cast<const void*>(p.bias + col) : qg_byte_rows.b[0];
        if (g == 3) src = p.scales + (size_t)min(col, N - 1) * p.scale_stride;
      }
      request_dword(src, (unsigned)(uintptr_t)((__attribute__((address_space(3))) int*)ep_s));
    }
  };

  // K slices are dealt to the waves rotated from workgroup to workgroup (qg_stream_slice): unrotated the workgroups of an XCD
  // would all hit the same L2 channel at the same time
  // (4-bit weights come in pairs of k blocks, so their slices hold an even number of blocks)
  // (ksplit > 1: this workgroup owns slice blockIdx.z of K, whole k blocks, an even number of them for 4-bit weights)
  // (plain shifts and additions up to the first loads: everything in front of them is latency)
  const int blocks = B4 ? (int)((unsigned)(K + 2 * QG_FRAG_K - 1) / (2 * QG_FRAG_K) * 2) : (int)((unsigned)(K + QG_FRAG_K - 1) / QG_FRAG_K);  // that hold data
  const int ks_begin = min(blocks, (int)blockIdx.z * ks_per), ks_end = min(blocks, ks_begin + ks_per);
  const int ks_len = ks_end - ks_begin;
  const int per = B4 ? (int)((unsigned)(ks_len + 2 * NWAVES - 1) / (2 * NWAVES) * 2) : (int)((unsigned)(ks_len + NWAVES - 1) / NWAVES);
  const int kb_begin = min(ks_end, ks_begin + qg_stream_slice(wave, blockIdx.x, NWAVES) * per);
  const int kb_end = min(ks_end, kb_begin + per);

  // outlier split: the entry offsets of all of this wave's batches, one per lane (batch b: lanes b and b+1), are
  // requested before anything else so that no batch waits for an offset before it can ask for its entries
  int sp_offs[CPW];
  if (B4 && kb_begin < kb_end) {
#pragma unroll
    for (int c = 0; c < CPW; ++c) sp_offs[c] = p.sp_ptr[(size_t)(nb16 + c) * kb64 + min(kb_begin + BATCH * lane, kb_end)];
  }

  v4i acc[MB][CPW];
  unsigned rs[MB];  // sums of raw uint8 bytes (K padding reads as 0x80)
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int c = 0; c < CPW; ++c) acc[mb][c] = (v4i){0, 0, 0, 0};
    rs[mb] = 0;
  }
  // 8-bit: one 1 KiB fragment per k block, 16 bytes per lane.  4-bit: one 1 KiB unit per PAIR of k blocks, 16 bytes
  // per lane (8 for each block), so that a request moves as many bytes as in the 8-bit layout.
  const int8_t* bcol = Bp + (size_t)nb16 * QG_FRAG_BYTES;  // wave-uniform; the lane's 16 bytes are at + lane * 16
  const unsigned lane16 = lane * 16;
  const size_t b_step = (size_t)nb16_total * QG_FRAG_BYTES;  // one slab (8-bit: 64 deep, 4-bit: 128 deep) of the packed buffer

  // per-lane byte offsets of the NREQ activation requests of a batch; with them the
  // request address is a wave-uniform base plus a register that is never the target of a load, so issuing
  // the requests never has to wait for loads in flight
  unsigned a_off[NREQ];
  // at most a quarter of the block's rows exist: only they are requested (what LDS holds in place of the others reaches only
  // accumulators that are never stored)
  const bool few = SRC == SRC_U8 && NREQ % 4 == 0 && M - m_base <= ROWS / 4;
  constexpr int FEW = NREQ / 4 > 0 ? NREQ / 4 : 1;
  // SRC_CONV: of the piece a lane requests for row block mb: byte offset of its pixel at tap (0, 0), channel slice 0 (may
  // be negative) and the taps of that pixel that lie inside the image; wave-uniform: the tap of the next k block
  int cv_pix[MB];
  unsigned cv_mask[MB];
  int cv_cc = 0, cv_kw = 0, cv_kh = 0;  // (SRC_CONV16: per lane, of the piece it requests; cv_cc in pieces)
  const int cv_nc = CONV ? p.cv_Cin / (SRC == SRC_CONV16 ? 16 : QG_FRAG_K) : 1;  // k blocks (pieces) per tap
  const int cv_wraps = SRC == SRC_CONV16 ? (4 + cv_nc - 1) / cv_nc : 0;  // taps that four pieces cross at most
  const uint8_t* const cv_azp_row = qg_byte_rows.b[CONV ? p.cv_azp : 0];
  const uint8_t* const pad_row = qg_byte_rows.b[128];
  if (CONV) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int r = mb * 16 + (lane >> 2);
      const int m = min(m_base + r, M - 1);
      const int wo = m % p.cv_Wo, t = m / p.cv_Wo;
      const int ho = t % p.cv_Ho, n = t / p.cv_Ho;
      const int h0 = ho * p.cv_stride - p.cv_pad, w0 = wo * p.cv_stride - p.cv_pad;
      // the lane's 16 bytes land at piece lane % 4 of its row's 64-byte block; that place holds logical piece (lane % 4) ^ (row / 4 % 4)
      cv_pix[mb] = ((n * p.cv_H + h0) * p.cv_W + w0) * p.cv_pix + (SRC == SRC_CONV ? (((lane & 3) ^ (lane >> 4)) & 3) << 4 : 0);
      // taps kw of [lo, hi) lie inside a row of the image: their bits once, shifted to each kh inside it (tap by tap, four compares
      // each, the 25 taps of 15 x 14 x 17 x 64 -> 64 cost 1.8 us of 7.1, serial before the first request)
      const int lo = w0 < 0 ? -w0 : 0, hi = p.cv_W - w0 < p.cv_S ? p.cv_W - w0 : p.cv_S;
      const unsigned row = hi > lo ? (unsigned)((1ull << hi) - (1ull << lo)) : 0u;
      cv_mask[mb] = 0;
      for (int kh = 0; kh < p.cv_R; ++kh)
        if ((unsigned)(h0 + kh) < (unsigned)p.cv_H) cv_mask[mb] |= row << (kh * p.cv_S);
    }
    const int at = SRC == SRC_CONV16 ? kb_begin * 4 + (((lane & 3) ^ (lane >> 4)) & 3) : kb_begin;
    const int tap = at / cv_nc;
    cv_cc = at - tap * cv_nc;
    cv_kh = tap / p.cv_S;
    cv_kw = tap - cv_kh * p.cv_S;
  } else {
#pragma unroll
    for (int jj = 0; jj < NREQ; ++jj) {
      const int r = jj * RPR + lane / NCHUNK;
      a_off[jj] = (unsigned)min(m_base + r, M - 1) * (unsigned)lda + ((unsigned)((lane ^ r) & (NCHUNK - 1)) << 4);
    }
  }
  // SRC_U8: the last 16 bytes of row `lane` (K >= 16)
  bool cut = false;  // (uniform) this wave has the chunk that K cuts
  v4i row_end;
  auto load_row_end = [&]() {
    cut = SRC == SRC_U8 && !WHOLE && (K & 15) != 0 && kb_end == blocks;
    if (cut) {
      const uint8_t* const row = A + (size_t)min(m_base + lane % ROWS, M - 1) * lda;
      if (K >= 16)
        row_end = *reinterpret_cast<const qg_v4i_unaligned*>(row + (K - 16));
      else
        row_end = qg_load_a_chunk(row, K, false);
    }
  };

  // Weight requests of one batch: 16 bytes per lane each, kept RAW (the 4-bit units are widened only
  // when they are consumed, so that nothing waits for them before the activations have been requested too).
  constexpr int NLOAD = (B4 ? BATCH / 2 : BATCH) * CPW;
  static_assert(!B4 || BATCH % 2 == 0, "4-bit weights are fetched in pairs of k blocks");
  // (every element is loaded unconditionally -- blocks past the end of the slice re-read its last block and are
  // never used -- so that the loaded registers are plain values and no copy has to wait for them)
  const int8_t* wptr = bcol + (size_t)(B4 ? kb_begin >> 1 : kb_begin) * b_step;  // B4: kb_begin and kb_end are even
  auto load_w = [&](int kb0, v4i (&raw)[NLOAD]) {  // batch by batch
    constexpr int STEP = B4 ? 2 : 1;
#pragma unroll
    for (int i = 0; i < NLOAD / CPW; ++i) {
#pragma unroll
      for (int c = 0; c < CPW; ++c) raw[i * CPW + c] = *reinterpret_cast<const v4i*>(wptr + c * QG_FRAG_BYTES + lane16);  // (adjacent KiBs)
      wptr += WHOLE || kb0 + (i + 1) * STEP < kb_end ? b_step : (size_t)0;
    }
  };
  auto operand = [&](const v4i (&raw)[NLOAD], int j, int c) -> v4i {
    if (!B4) return raw[j * CPW + c];
    const v4i w = raw[(j >> 1) * CPW + c];
    const unsigned lo = (unsigned)((j & 1) ? w.z : w.x), hi = (unsigned)((j & 1) ? w.w : w.y);
    return (v4i){(int)(lo & 0x0F0F0F0Fu), (int)((lo >> 4) & 0x0F0F0F0Fu), (int)(hi & 0x0F0F0F0Fu),
                 (int)((hi >> 4) & 0x0F0F0F0Fu)};
  };

  unsigned char* const region0 = smem + wave * WAVE_LDS;
  const unsigned region0_lds = (unsigned)(uintptr_t)((__attribute__((address_space(3))) unsigned char*)region0);

  // ROWS rows x ROWB bytes of A: NREQ requests of RPR whole rows into this wave's region `buf`, chunk c of
  // row r stored at chunk c ^ r so that the operand-order reads below are bank-conflict free.  Whole rows of BATCH k blocks are
  // requested even when the wave's part of K ends earlier: the surplus is not consumed.
  auto request_rows = [&](int kb, int buf) {
    const unsigned dst = region0_lds + buf * REGION;
    if constexpr (SRC == SRC_CONV16) {
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        const bool in_k = cv_kh < p.cv_R;
        const unsigned tapbit = in_k ? 1u << (cv_kh * p.cv_S + cv_kw) : 0u;
        const int toff = (cv_kh * p.cv_W + cv_kw) * p.cv_pix + cv_cc * 16;
        const uint8_t* const other = in_k ? cv_azp_row : pad_row;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          request_a64((cv_mask[mb] & tapbit) != 0 ? A + (cv_pix[mb] + toff) : other, dst + (j * MB + mb) * 1024);
        cv_cc += 4;
        for (int i = 0; i < cv_wraps; ++i)
          if (cv_cc >= cv_nc) {
            cv_cc -= cv_nc;
            if (++cv_kw == p.cv_S) cv_kw = 0, ++cv_kh;
          }
      }
    } else if constexpr (SRC == SRC_CONV) {
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        // (wave-uniform) a k block past K -- the zero padding of the packed weights -- is staged as 0x80 bytes like
        // all K padding, a tap outside the image as theta_A bytes
        const bool in_k = cv_kh < p.cv_R;
        const unsigned tapbit = in_k ? 1u << (cv_kh * p.cv_S + cv_kw) : 0u;
        const int toff = (cv_kh * p.cv_W + cv_kw) * p.cv_pix + cv_cc * QG_FRAG_K;
        const uint8_t* const other = in_k ? cv_azp_row : pad_row;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          request_a64((cv_mask[mb] & tapbit) != 0 ? A + (cv_pix[mb] + toff) : other, dst + (j * MB + mb) * 1024);
        if (++cv_cc == cv_nc) {
          cv_cc = 0;
          if (++cv_kw == p.cv_S) cv_kw = 0, ++cv_kh;
        }
      }
    } else {
      const uint8_t* const a_base = A + (size_t)kb * QG_FRAG_K;  // wave-uniform
      if (WHOLE || (kb + BATCH) * QG_FRAG_K <= K) {
        if (few) {
#pragma unroll
          for (int jj = 0; jj < FEW; ++jj) request_a(a_base, a_off[jj], dst + jj * 1024);
        } else {
#pragma unroll
          for (int jj = 0; jj < NREQ; ++jj) request_a(a_base, a_off[jj], dst + jj * 1024);
        }
      } else {
        int l = lane;
        asm volatile("" : "+v"(l));  // (opaque: what the requests of this rare batch need is not kept in registers for it)
#pragma unroll
        for (int jj = 0; jj < NREQ; ++jj) {
          if (few && jj >= FEW) break;
          const int r = jj * RPR + l / NCHUNK, k0 = kb * QG_FRAG_K + (((l ^ r) & (NCHUNK - 1)) << 4);
          request_a64(k0 + 16 <= K ? a_base + a_off[jj] : pad_row, dst + jj * 1024);
        }
      }
    }
  };
  // the chunk that K cuts, over what its request left there
  auto put_row_end = [&](int kb, int buf) {
    if (WHOLE) return;
    const int c = (K >> 4) - kb * (QG_FRAG_K / 16);  // its place in the batch
    if (cut && c < NCHUNK) {
      const v4i v = K >= 16 ? qg_row_end_chunk(row_end, K & 15) : row_end;
      const int r = lane % ROWS;
      if (lane < ROWS) *reinterpret_cast<v4i*>(region0 + buf * REGION + r * ROWB + (((c ^ r) & (NCHUNK - 1)) << 4)) = v;
      asm volatile("" ::: "memory");  // (the operand reads below are of other lanes' chunks; LDS operations of a wave run in order)
    }
  };
  // fp32 rows: four floats per lane, a load is 4 rows x 64 floats of one k block.  Only the blocks that the wave consumes and the
  // rows that exist, GRP loads in flight.
  auto convert_rows = [&](int kb) {
    const float* const Af = reinterpret_cast<const float*>(A);
    constexpr int GRP = 8;
    typedef float v4f __attribute__((ext_vector_type(4)));
    typedef v4f v4f_any __attribute__((aligned(4)));
    const int nblk = min(BATCH, kb_end - kb), groups = (min(ROWS, M - m_base) + 3) / 4;
    const int sh = groups <= 1 ? 0 : 32 - __builtin_clz(groups - 1), total = nblk << sh;  // load i: block i >> sh, rows 4 (i mod 2^sh) ...
    int l = lane;
    asm volatile("" : "+v"(l));  // (opaque: nothing of this is kept in registers across the batches)
    const int q = l & 15;        // this lane's dword of the block
    // 0: a batch inside K; 1: K ends in it (the last four floats of the row for whatever begins past them, the bytes shifted into
    // place: 0.95 of the time with four loads per lane, K off 64); 2: K < 4, float by float
    auto convert = [&](auto form) {
      constexpr bool INSIDE = decltype(form)::value == 0;
#pragma unroll 1
      for (int t0 = 0; t0 < total; t0 += GRP) {
        v4f v[GRP];
#pragma unroll
        for (int t = 0; t < GRP; ++t) {
          const int i = min(t0 + t, total - 1), r = (i & ((1 << sh) - 1)) * 4 + (l >> 4), k = (kb + (i >> sh)) * QG_FRAG_K + q * 4;
          const float* const row = Af + (size_t)min(m_base + r, M - 1) * lda;
          if (INSIDE) {
            v[t] = *reinterpret_cast<const v4f_any*>(row + k);
          } else if (decltype(form)::value == 1) {
            const int at = min(k, K - 4);
            v[t] = *reinterpret_cast<const v4f_any*>(row + at);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[t][e] = row[min(k + e, K - 1)];
          }
        }
#pragma unroll
        for (int t = 0; t < GRP; ++t) {
          const int i = min(t0 + t, total - 1), j = i >> sh, r = (i & ((1 << sh) - 1)) * 4 + (l >> 4);
          unsigned d = 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) d = qg_quantize_pack(v[t][e], p.q_inv, p.q_zp, e, d);
          if (!INSIDE) {
            if (decltype(form)::value == 1) d >>= 8 * min(max((kb + j) * QG_FRAG_K + q * 4 - (K - 4), 0), 3);
            const int nv = min(max(K - (kb + j) * QG_FRAG_K - q * 4, 0), 4);
            const unsigned keep = nv == 4 ? 0xFFFFFFFFu : (1u << (8 * nv)) - 1u;
            d = (d & keep) | (0x80808080u & ~keep);
          }
          *reinterpret_cast<unsigned*>(region0 + r * ROWB + (((4 * j + (q >> 2)) ^ r) & (NCHUNK - 1)) * 16 + (q & 3) * 4) = d;
        }
      }
    };
    if ((kb + nblk) * QG_FRAG_K <= K)
      convert(std::integral_constant<int, 0>{});
    else if (K >= 4)
      convert(std::integral_constant<int, 1>{});
    else
      convert(std::integral_constant<int, 2>{});
    asm volatile("" ::: "memory");
  };

  // outlier split: a batch's entries are one run per fragment column; the first 64 are requested one per lane (always exactly one
  // request, clamped into the buffer, so that the waits can count it)
  struct entries {
    int at[CPW], n[CPW], first[CPW];
  };
  auto request_entries = [&](int b, entries& e) {
    if (B4) {
#pragma unroll
      for (int c = 0; c < CPW; ++c) {  // at most 32 batches per wave: K <= 32768 gives 128 blocks to each of four waves, four a batch
        e.at[c] = __builtin_amdgcn_readlane(sp_offs[c], b);
        e.n[c] = __builtin_amdgcn_readlane(sp_offs[c], b + 1) - e.at[c];
        e.first[c] = p.sp_entries[min(e.at[c] + lane, max(p.sp_total, 1) - 1)];
      }
    }
  };

  auto consume = [&](int kb, int buf, const v4i (&cur)[NLOAD], const entries& ent) {
    unsigned char* const region = region0 + buf * REGION;
    // many outliers: the batch's entries beyond the first 64, four loads at a time, the first four in front of the dense products
    // where registers allow it
    constexpr bool EARLY = CPW == 1 || NWAVES < 16;
    int more[CPW][4];
    auto load_more = [&](int c, int i0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) more[c][u] = p.sp_entries[ent.at[c] + min(i0 + 64 * u + lane, ent.n[c] - 1)];
    };
    if (B4 && EARLY) {
#pragma unroll
      for (int c = 0; c < CPW; ++c)
        if (ent.n[c] > 64) load_more(c, 64);
    }
    v4i af[MB][BATCH];
    // (chunk 4 j + g of row r lies at (4 j + g) ^ r: the place of j = 0 with j turned into it.  Opaque, or the compiler keeps all
    // the places in registers across the batches.)
    int at = CONV ? ml * QG_FRAG_K + (((g ^ (ml >> 2)) & 3) << 4) : ml * ROWB + (((g ^ ml) & (NCHUNK - 1)) << 4);
    asm volatile("" : "+v"(at));
#pragma unroll
    for (int j = 0; j < BATCH; ++j)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        if (CONV)  // [k block][row block][row][piece ^ (row / 4 % 4)]
          af[mb][j] = *reinterpret_cast<const v4i*>(region + at + (j * MB + mb) * 1024);
        else  // (rows 16 further: bit 4 of the row is turned into the chunk too)
          af[mb][j] = *reinterpret_cast<const v4i*>(region + mb * (16 * ROWB) + (at ^ (((4 * j) ^ (mb * 16 & (NCHUNK - 1))) << 4)));
      }
    auto dense = [&](int j) {
      v4i w[CPW];
#pragma unroll
      for (int c = 0; c < CPW; ++c) w[c] = operand(cur, j, c);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        rs[mb] = __builtin_amdgcn_sad_u8(af[mb][j].x, 0u, rs[mb]);
        rs[mb] = __builtin_amdgcn_sad_u8(af[mb][j].y, 0u, rs[mb]);
        rs[mb] = __builtin_amdgcn_sad_u8(af[mb][j].z, 0u, rs[mb]);
        rs[mb] = __builtin_amdgcn_sad_u8(af[mb][j].w, 0u, rs[mb]);
        af[mb][j] = af[mb][j] ^ (int)0x80808080;
#pragma unroll
        for (int c = 0; c < CPW; ++c) acc[mb][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[c], af[mb][j], acc[mb][c], 0, 0, 0);
      }
    };
    if (WHOLE || kb + BATCH <= kb_end) {
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        dense(j);
        if (B4) __builtin_amdgcn_sched_barrier(0);  // (or all the widened weights of the batch are in registers at once)
      }
    } else {
#pragma unroll
      for (int j = 0; j < BATCH; ++j)
        if (kb + j < kb_end) dense(j);
    }
    if (B4) {
      // sparse term of this batch.  The lanes hand each other bytes through the wave's region: its LDS operations run in order
      // -- the reads above, the zeros, the bytes, the reads --, and the empty statements keep the compiler, which looks at one
      // lane at a time, from reordering them or from taking a lane's own zeros for what it will read.
#pragma unroll
      for (int c = 0; c < CPW; ++c) {
        if (ent.n[c] <= 0) continue;
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < BATCH; ++j) *reinterpret_cast<v4i*>(region + j * QG_FRAG_BYTES + lane * 16) = (v4i){0, 0, 0, 0};
        asm volatile("" ::: "memory");
        auto scatter = [&](int e) {
          const int kk = (e & 0x7FFF) - kb * QG_FRAG_K, slot = (e >> 16) & 15;
          region[(kk >> 6) * QG_FRAG_BYTES + ((((kk >> 4) & 3) << 4) + slot) * 16 + (kk & 15)] = (unsigned char)(e >> 24);
        };
        if (lane < ent.n[c]) scatter(ent.first[c]);
        for (int i0 = 64; i0 < ent.n[c]; i0 += 4 * 64) {
          int e[4];
          if (!EARLY) load_more(c, i0);
#pragma unroll
          for (int u = 0; u < 4; ++u) e[u] = more[c][u];
          if (EARLY && i0 + 4 * 64 < ent.n[c]) load_more(c, i0 + 4 * 64);
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (i0 + 64 * u + lane < ent.n[c]) scatter(e[u]);
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int j = 0; j < BATCH; ++j)
          if (kb + j < kb_end) {
            const v4i sf = *reinterpret_cast<const v4i*>(region + j * QG_FRAG_BYTES + lane * 16);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) acc[mb][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(sf, af[mb][j], acc[mb][c], 0, 0, 0);
          }
        asm volatile("" ::: "memory");  // these reads stay in front of the next requests into the same region
      }
    }
    asm volatile("" ::: "memory");  // ... like the fragment reads
  };

  // fp32 activations with a place for the quantized rows: they are stored from LDS when the batch has been consumed, so that no wait
  // for loads in front of the MFMAs waits for the stores too (over 8900 drawn calls two launches take 1.109 times the better of one
  // and two; 1.079 with the stores beside the conversion, 1.20 with no copy at all).  The column blocks store two k blocks, whole
  // cache lines, each in turn: a power of two of them without the last, which may have returned for want of columns.
  auto copy_rows = [&](int kb) {
    if constexpr (SRC == SRC_F32) {
      if (p.q_copy == nullptr) return;
      const int turns = gridDim.x > 2 ? (1 << (31 - __builtin_clz(gridDim.x - 1))) - 1 : 0;
      const int nblk = min(BATCH, kb_end - kb), rows = min(ROWS, M - m_base);
      int l = lane;
      asm volatile("" : "+v"(l));
      for (int j = 0; j < nblk; ++j) {
        if ((((kb + j) >> 1) & turns) != (int)blockIdx.x) continue;
        for (int r = l >> 2; r < rows; r += 16) {
          const v4i v = *reinterpret_cast<const v4i*>(region0 + r * ROWB + ((((4 * j + (l & 3)) ^ r) & (NCHUNK - 1)) << 4));
          const unsigned w[4] = {(unsigned)v[0], (unsigned)v[1], (unsigned)v[2], (unsigned)v[3]};
          const int k = (kb + j) * QG_FRAG_K + (l & 3) * 16;
          qg_store_columns(p.q_copy + (size_t)(m_base + r) * p.q_ldq + k, w, K - k);
        }
      }
      asm volatile("" ::: "memory");
    }
  };

  // Two register sets alternate.  A batch's weights are requested one batch ahead, its activations with them (DB) or at its
  // start; requests complete in order, so "at most the next batch's outstanding" means that this one has arrived.
  const int nbatch = kb_begin < kb_end ? (kb_end - kb_begin + BATCH - 1) / BATCH : 0;
  auto step = [&](int b, int buf, v4i (&cur)[NLOAD], v4i (&nxt)[NLOAD], entries& ent, entries& ent_nxt) {
    const int kb = kb_begin + b * BATCH;
    const bool has_next = b + 1 < nbatch;
    if constexpr (SRC == SRC_F32) {
      convert_rows(kb);
      if (b == 0) request_ep();
      if (has_next) load_w(kb + BATCH, nxt);
    } else if constexpr (DB) {
      if (has_next) {
        load_w(kb + BATCH, nxt);
        request_rows(kb + BATCH, buf ^ 1);
        request_entries(b + 1, ent_nxt);
        asm volatile("" ::: "memory");
        if (few)
          wait_vm<NLOAD + FEW + (B4 ? CPW : 0)>();
        else
          wait_vm<NLOAD + NREQ + (B4 ? CPW : 0)>();
      } else {
        wait_vm<0>();
      }
    } else {
      if (b != 0) request_rows(kb, buf);
      asm volatile("" ::: "memory");
      if (has_next) {
        load_w(kb + BATCH, nxt);
        wait_vm<NLOAD>();
      } else {
        wait_vm<0>();
      }
    }
    put_row_end(kb, buf);
    consume(kb, buf, cur, ent);
    if (has_next) copy_rows(kb);
  };
  if constexpr (ONE) {
    v4i w0[NLOAD];
    load_w(kb_begin, w0);
    request_rows(kb_begin, 0);
    request_ep();
    asm volatile("" ::: "memory");
    wait_vm<0>();
    consume(kb_begin, 0, w0, entries());
  } else if (nbatch > 0) {
    v4i w0[NLOAD], w1[NLOAD];
    entries e0, e1;
    if constexpr (B4) {  // (the offsets of the entries are waited for by the count of the loads behind them: no requests among those)
      request_rows(kb_begin, 0);
      load_row_end();
      load_w(kb_begin, w0);
      request_entries(0, e0);
      request_ep();
    } else {
      load_w(kb_begin, w0);
      if (SRC != SRC_F32) {
        request_rows(kb_begin, 0);
        load_row_end();
        request_ep();
      }
    }
    asm volatile("" ::: "memory");
    step(0, 0, w0, w1, e0, e1);
    for (int b = 1; b < nbatch; b += 2) {
      step(b, DB ? 1 : 0, w1, w0, e1, e0);
      if (b + 1 < nbatch) step(b + 1, 0, w0, w1, e0, e1);
    }
  } else {
    request_ep();
  }

  wait_vm<0>();  // the output pipeline's constants (the waves without a part in it read what is there)
  if (nbatch > 0) copy_rows(kb_begin + (nbatch - 1) * BATCH);
  const int* const ep_r = wave < MB * CPW ? ep_s : rsp;
  const v4i ep_co = *reinterpret_cast<const v4i*>(ep_r + 4 * g), ep_bz = *reinterpret_cast<const v4i*>(ep_r + 16 + 4 * g);
  const v4i ep_bias = *reinterpret_cast<const v4i*>(ep_r + 32 + 4 * g);
  const float4 ep_sc4 = *reinterpret_cast<const float4*>(ep_r + 48 + 4 * g);
  const float ep_sc[4] = {ep_sc4.x, ep_sc4.y, ep_sc4.z, ep_sc4.w};

  // ---- combine the waves' K-slices through LDS (a wave's fragment reads of its region are complete: the MFMAs consumed them)
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int c = 0; c < CPW; ++c) reinterpret_cast<v4i*>(region0)[(mb * CPW + c) * 64 + lane] = acc[mb][c];
    // the four lanes (ml, g = 0..3) of a row hold its byte sums over different k: add them with two lane swaps
    // (v_permlane32_swap / v_permlane16_swap; a shuffle through the LDS crossbar costs about 100 cycles each)
    const unsigned v = rs[mb];
    const auto h = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    const unsigned v2 = h[0] + h[1];
    const auto q = __builtin_amdgcn_permlane16_swap(v2, v2, false, false);
    if (g == 0) rsp[((mb * 16 + ml) * NWAVES) + wave] = (int)(q[0] + q[1]);  // [mb][row][wave]: the reader takes a row's 16 sums in four reads
  }
  __syncthreads();
  if (wave >= MB * CPW) return;
  const int mb = red_mb;
  v4i sum = (v4i){0, 0, 0, 0};
  int rsum = -128 * (ks_len * QG_FRAG_K);  // every staged byte (padding included) is 128 above its int8 value
  {
    // every read is issued before the first sum (a sum per read would serialise on the LDS latency, 16 times over)
    static_assert(NWAVES % 4 == 0, "row sums are fetched four waves at a time");
    v4i t[NWAVES], tr[NWAVES / 4];
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) t[w] = reinterpret_cast<const v4i*>(smem + w * WAVE_LDS)[(mb * CPW + red_c) * 64 + lane];
#pragma unroll
    for (int w = 0; w < NWAVES / 4; ++w) tr[w] = reinterpret_cast<const v4i*>(rsp + (mb * 16 + ml) * NWAVES)[w];
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) sum += t[w];
#pragma unroll
    for (int w = 0; w < NWAVES / 4; ++w) rsum += tr[w].x + tr[w].y + tr[w].z + tr[w].w;
  }
  if (B4) {
    // A_s B = (A_s U - 8 rowsum(A_s)) + A_s B_sparse
#pragma unroll
    for (int r = 0; r < 4; ++r) sum[r] -= 8 * rsum;
  }

  // ---- K split across workgroups: hand the partial tile in, the last slice to arrive carries on
  if (ksplit > 1) {
    // one counter per (row block of 16, fragment column)
    const int unit = (((int)blockIdx.y * (int)gridDim.x + (int)blockIdx.x) * CPW + red_c) * MB + mb;
    int* cnt = p.ws_cnt + unit;
    int* slots = p.ws_slots + (size_t)unit * ksplit * SLOT_INTS;
    int* mine = slots + (size_t)blockIdx.z * SLOT_INTS;
#pragma unroll
    for (int r = 0; r < 4; ++r) __hip_atomic_store(mine + lane * 4 + r, sum[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (g == 0) __hip_atomic_store(mine + 256 + ml, rsum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the write-through stores above have been acknowledged
    int ticket = 0;
    if (lane == 0) ticket = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ticket = __builtin_amdgcn_readfirstlane(ticket);
    if (ticket != ksplit - 1) return;
    asm volatile("" ::: "memory");
    // every other slice's stores were acknowledged before it took its ticket; add all slots in slice order
    sum = (v4i){0, 0, 0, 0};
    rsum = 0;
#pragma unroll 4  // the loads of four slots are in flight together
    for (int ss = 0; ss < ksplit; ++ss) {
      const int* theirs = slots + (size_t)ss * SLOT_INTS;
#pragma unroll
      for (int r = 0; r < 4; ++r) sum[r] += __hip_atomic_load(theirs + lane * 4 + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      rsum += __hip_atomic_load(theirs + 256 + ml, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane == 0) __hip_atomic_store(cnt, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next call
  }

  // ---- output pipeline; lane (ml, u = g) holds row m_base+mb*16+ml, 4 consecutive columns
  const int row = m_base + mb * 16 + ml;
  if (row >= M || c0 >= N) return;
  if (MODE == QG_MODE_REQUANT) {
    unsigned out = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int x = sum[r] + ep_bias[r] - p.a_zp_m128 * ep_co[r] - ep_bz[r] * rsum;
      out |= (unsigned)qg_requant_one(x, ep_sc[r], p.clamp_lo, p.clamp_hi, p.c_zp) << (8 * r);
    }
    uint8_t* dst = p.C + (size_t)row * p.ldc + c0;
    if (p.c_vec && c0 + 4 <= N) {
      // a small output goes out write-through: the end of the kernel then finds no dirty lines to write back
      // (measured: 0.3 us of a 5 us launch)
      if (p.c_wt)
        __hip_atomic_store(reinterpret_cast<unsigned*>(dst), out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      else
        *reinterpret_cast<unsigned*>(dst) = out;
    } else {
      qg_store_columns(dst, {out, 0, 0, 0}, min(N - c0, 4));
    }
  } else if (MODE == QG_MODE_DEQUANT) {
    float out[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int x = sum[r] + ep_bias[r] - p.a_zp_m128 * ep_co[r] - ep_bz[r] * rsum;
      out[r] = qg_dequant_one(x, ep_sc[r], p.relu_lo);
    }
    float* dst = p.Cf + (size_t)row * p.ldc + c0;
    if (p.c_vec && c0 + 4 <= N) {
      *reinterpret_cast<float4*>(dst) = make_float4(out[0], out[1], out[2], out[3]);
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (c0 + r < N) dst[r] = out[r];
    }
  } else {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int col = c0 + r;
      if (col < N) p.C32[(size_t)row * p.ldc + col] = sum[r] + 128 * (ep_co[r] + K * ep_bz[r]);
    }
    if (p.rowsum_out != nullptr && nb16 + red_c == 0 && g == 0) p.rowsum_out[row] = rsum + 128 * K;
  }
}

template <int MODE, int MB, int NWAVES, int BATCH, int CPW, bool B4, int SRC, bool DB, bool WHOLE = false>
hipError_t launch(const qg_gemm_args& a, hipStream_t s) {
  constexpr int SMEM = NWAVES * (MB * 16) * (BATCH * QG_FRAG_K) * (DB ? 2 : 1) + NWAVES * MB * 16 * (int)sizeof(int) + MB * CPW * 256;
  static_assert(SMEM <= 160 * 1024, "LDS of a CU");
  const int mblocks = (a.M + MB * 16 - 1) / (MB * 16);
  if (mblocks > 65535 || a.ksplit < 1 || a.ksplit > 65535) return hipErrorInvalidValue;
  if (a.ksplit > 1 && (a.ws_cnt == nullptr || a.ws_slots == nullptr)) return hipErrorInvalidValue;
  constexpr auto fn = qg_gemm_skinny_kernel<MODE, MB, NWAVES, BATCH, CPW, B4, SRC, DB, WHOLE>;
  hipError_t e = qg_allow_smem<fn>(SMEM);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fn, dim3(((a.N + 31) / 32) * 2 / CPW, mblocks, a.ksplit), dim3(NWAVES * 64), SMEM, s, a.A, a.Bp, a.M, a.N, a.K,
                     a.kb64, a.nb16, a.lda, a.ks_per, a.ksplit, a);
  return hipGetLastError();
}
template <int MODE, bool B4, int SRC>
hipError_t launch_form(const qg_gemm_args& a, int kernel, hipStream_t s) {
  constexpr bool DB = SRC != SRC_F32;
  if (kernel < QG_KERNEL_SKINNY16 || kernel > QG_KERNEL_SKINNY64) return hipErrorInvalidValue;
  const int blocks = (a.K + QG_FRAG_K - 1) / QG_FRAG_K, kb = blocks < a.ks_per ? blocks : a.ks_per;
  const int rows = 16 << (kernel - QG_KERNEL_SKINNY16);
  const long long sb = (long long)((a.N + 31) / 32) * ((a.M + rows - 1) / rows) * a.ksplit;
  const qg_stream_build f = qg_stream_build_of(rows, kb, sb, a.M, B4);
  if constexpr (SRC == SRC_U8 && !B4) {
    // Whole batches in every wave of every slice.  One batch: 13 x 3328 x 1024 2.67 us on the build for any K, 2.46 so (four waves), 16 x 640
    // x 2048 2.82 and 2.61 (eight), 80 x 1536 x 2048 3.52 and 3.43 (two columns; 12 shapes 0.96 to 1.01 of the loop over batches, which
    // holds two regions); several ahead of each other: 8 x 4832 x 4096 5.61 and 5.47, 16 x 14048 x 4096 10.50 and 10.42.
    // Four waves with several batches are not faster so (M up to 4 and a long K: 1.00 to 1.04).
    if (rows == 16 && kb * a.ksplit == blocks && qg_stream_whole(f, kb, a.K)) {
      if (qg_stream_far(f, kb, sb)) return launch<MODE, 1, 4, 8, 2, B4, SRC, false, true>(a, s);
      if (f.columns == 2 && kb == f.waves * f.batch) return launch<MODE, 1, 8, 4, 2, B4, SRC, false, true>(a, s);
      if (f.columns == 2) return launch<MODE, 1, 8, 4, 2, B4, SRC, true, true>(a, s);
      if (f.waves == 4) return launch<MODE, 1, 4, 4, 1, B4, SRC, false, true>(a, s);
      if (f.waves == 8) return launch<MODE, 1, 8, 4, 1, B4, SRC, false, true>(a, s);
      return launch<MODE, 1, 16, 4, 1, B4, SRC, false, true>(a, s);
    }
  }
  if constexpr (B4) {
    if (f.waves == 4 && f.batch == 2) {
      if (rows == 16) return launch<MODE, 1, 4, 2, 1, B4, SRC, DB>(a, s);
      return rows == 32 ? launch<MODE, 2, 4, 2, 1, B4, SRC, DB>(a, s) : launch<MODE, 4, 4, 2, 1, B4, SRC, DB>(a, s);
    }
  }
  if constexpr (SRC == SRC_F32) {
    // fp32 rows: the conversion is what a wave spends its time on, nothing is requested ahead, so a long K takes all the waves there are.
    // 64 rows: 42 x 3714 x 3840 21.8 us with eight, 18.7 so; 68 shapes of up to 128 super-blocks 0.82 to 0.96, K of 2560 1.02 to 1.05; up to
    // 16 k blocks a wave has one batch either way.  16 rows: 117 x 64 x 7680 13.3 us and 11.1, 46 shapes 0.80 to 1.00; from 65 to 95 k blocks
    // 0.93 to 1.08, the second batch of sixteen waves half empty.
    if (rows == 64 && f.columns == 1 && kb > 16) return launch<MODE, 4, 16, 2, 1, B4, SRC, DB>(a, s);
    if (rows == 16 && f.columns == 1 && f.waves == 8 && kb >= 96) return launch<MODE, 1, 16, 4, 1, B4, SRC, DB>(a, s);
  }
  switch (rows * 10000 + f.waves * 100 + f.batch * 10 + f.columns) {
    case 160441: return launch<MODE, 1, 4, 4, 1, B4, SRC, DB>(a, s);
    case 160841: return launch<MODE, 1, 8, 4, 1, B4, SRC, DB>(a, s);
    case 160842: return launch<MODE, 1, 8, 4, 2, B4, SRC, DB>(a, s);
    case 161641: return launch<MODE, 1, 16, 4, 1, B4, SRC, B4>(a, s);  // (8-bit: one batch, nothing to request ahead)
    case 320841: return launch<MODE, 2, 8, 4, 1, B4, SRC, DB>(a, s);
    case 320842: return launch<MODE, 2, 8, 4, 2, B4, SRC, DB>(a, s);
    case 321621: return launch<MODE, 2, 16, 2, 1, B4, SRC, DB>(a, s);
    default: break;
  }
  if constexpr (SRC != SRC_CONV16) {  // (64 rows: the choice for 1 of 1536 drawn layers, and 2 % slower there)
    if (rows == 64)
      return f.columns == 2 ? launch<MODE, 4, 8, 2, 2, B4, SRC, DB>(a, s) : launch<MODE, 4, 8, 2, 1, B4, SRC, DB>(a, s);
  }
  if (rows == 64) return hipErrorInvalidValue;
  if constexpr (B4) {
    if (f.waves == 16 && f.columns == 2) return launch<MODE, 1, 16, 4, 2, B4, SRC, DB>(a, s);
  } else {
    if (f.waves == 4) return launch<MODE, 2, 4, 4, 2, B4, SRC, DB>(a, s);
    if (f.waves == 16) return launch<MODE, 2, 16, 4, 1, B4, SRC, false>(a, s);  // (LDS for one batch per wave)
  }
  return hipErrorInvalidValue;
}
template <bool B4>
hipError_t launch_mode(const qg_gemm_args& a, int mode, int kernel, hipStream_t s) {
  if (mode == QG_MODE_REQUANT) return launch_form<QG_MODE_REQUANT, B4, SRC_U8>(a, kernel, s);
  if (mode == QG_MODE_DEQUANT) return launch_form<QG_MODE_DEQUANT, B4, SRC_U8>(a, kernel, s);
  return launch_form<QG_MODE_ACC32, B4, SRC_U8>(a, kernel, s);
}

}  // namespace

// Dense convolution on the streaming kernels: few output pixels and a long K.  Cin % 16 == 0 (% 64 for the 64-row one), R*S <= 32.
hipError_t qg_launch_conv_skinny(const qg_gemm_args& a, int kernel, hipStream_t s) {
  if (a.sp_ptr != nullptr || a.cv_Cin % 16 != 0 || a.cv_R * a.cv_S > 32 || a.ksplit != 1) return hipErrorInvalidValue;
  return a.cv_Cin % QG_FRAG_K == 0 ? launch_form<QG_MODE_REQUANT, false, SRC_CONV>(a, kernel, s)
                                   : launch_form<QG_MODE_REQUANT, false, SRC_CONV16>(a, kernel, s);
}

// a.A points to fp32 activations (a.lda in floats, a.q_*: the quantization); mode: QG_MODE_REQUANT or QG_MODE_DEQUANT
hipError_t qg_launch_gemm_skinny_f32(const qg_gemm_args& a, int mode, int kernel, hipStream_t s) {
  if (a.sp_ptr != nullptr || mode == QG_MODE_ACC32) return hipErrorInvalidValue;
  return mode == QG_MODE_REQUANT ? launch_form<QG_MODE_REQUANT, false, SRC_F32>(a, kernel, s)
                                 : launch_form<QG_MODE_DEQUANT, false, SRC_F32>(a, kernel, s);
}

hipError_t qg_launch_gemm_skinny(const qg_gemm_args& a, int mode, int kernel, hipStream_t s) {
  // a.sp_ptr != null: Bp holds the 4-bit part of an outlier-split matrix
  return a.sp_ptr != nullptr ? launch_mode<true>(a, mode, kernel, s) : launch_mode<false>(a, mode, kernel, s);
}
