#!/usr/bin/env python3
"""Writes tile_loop_asm.inc: the software-pipelined main loop of the large-tile GEMM kernel as one
inline-asm string.

Why assembly: with one wave per SIMD (256 accumulator registers per wave) nothing but the order of the
instruction stream hides LDS and memory latency, and the compiler's scheduler clusters LDS reads, VALU
work and tile requests instead of spreading them behind the MFMAs.  Measured on MI355X, each
v_mfma_i32_32x32x32_i8 occupies the matrix pipe for 32 cycles, in whose shadow up to seven other
instructions of the same wave can issue for free; v_dot4 is NOT free (it shares the pipe), v_sad_u8 is.

Fixed register plan (all clobbered by the asm statement):
  v[160:175] A fragments set 0   v[176:191] B fragments set 0
  v[192:207] A fragments set 1   v[208:223] B fragments set 1
  v[224:227] row-sum accumulators (raw uint8 byte sums)
  v[228:231] per-lane byte offsets of the 4 A tile requests, v[232:235] of the 4 B tile requests
  v236/v237  per-lane LDS offsets of the A fragment for k-step 0 / 1, v238 of the B fragment
  v240/v241  LDS read addresses (stage base added)
  s84 xor mask, s[86:87] A request base, s[88:89] B request base, s90 loop counter, s91 LDS base of
  this wave's request slots, s92 LDS base, s99 bytes per 64-deep slab of packed B, s93 stage index, s96 request stage base, s97/s98 read
  stage bases (current / next), s94/s95 temporaries
m0 is written in front of every group of requests and is not among the clobbered registers: the compiler reserves it,
refuses it in a clobber list and sets it anew in front of each of its own uses.
Operands: 16 accumulators c0..c15 ("+a", acc[mb][nb] = c{4*mb+nb}), packed 64-bit VGPR inputs
av01 av23 bv01 bv23 ard brd, SGPR inputs aptr bptr kt ldsdma lds bstep, 64-bit VGPR outputs rs01 rs23.

Two configurations are generated from the same schedule: TM x TN = 4 x 4 blocks per wave (256 x 256 workgroup
tile, the plan above) and 2 x 2 (128 x 128 tile: 4 accumulators c0..c3, inputs av01 bv01 ard brd, output rs01,
fixed registers from v96, 16 KiB stages).  With only four MFMAs per k-step the LDS reads sit behind the first
two and the row sums and shifts of both A fragments behind the last two.  A third one, 2 x 4 blocks (128 x 256
tile: 8 accumulators, three 24 KiB stages so that two workgroups share a CU, fixed registers from v56, one more
SGPR input bofs = distance from a wave's A request slots to its B request slots), has eight MFMAs per k-step.

Fourth, the 2 x 2 loop for a set of only two waves (128 x 64 tile, four sets that split K, three 48 KiB stages of four k
tiles): A is requested by all eight waves together, 128 bytes = two tiles of a row at a time (the L1 looks up one line
per cycle whether 64 or 128 bytes of it are wanted: 55 against 86 bytes per cycle measured), into 16 KiB regions of 128
rows x 128 bytes that two sets share; a wave makes four requests of A and two of its set's B per step (inputs av23 and bofs
as well) and moves on by 256 bytes of A (ASTEP) and four slabs of B (bstep).  Rows are 128 bytes apart (A_BLOCK).

PAIR (4 x 4): A is requested 128 bytes of a row at a time -- two k tiles, one whole cache line --, one half of the
tile's rows per k tile.  Requesting 64 bytes per row and tile fetched every line twice: the other half had left the 32 KB
L1 by the time it was asked for (6.4 GB from the L2s instead of 4.3 at 8192^3), and this tile is limited by power, not by
issue.  A's LDS is a ring of six half buffers (rows 128 bytes apart, chunk c of row r at c ^ (r >> 1 & 7)), two of which
make the pair of tiles 2 P, 2 P + 1; B keeps its four stages behind them.  Tile t requests half t + 5 (rows of half
t + 5 & 1 of pair t + 5 >> 1) and B tile t + 4, so every wait is the one of the plain loop.  With an even number of tiles
the last tile that requests asks for half KT, which does not exist: the pointer is not advanced and the last pair comes
again, into a slot nobody reads.  With an odd number the last pair has 64 valid bytes per row: lanes whose chunk lies past
them ask for one 64 bytes earlier (afix: 64 or 0 for requests of even number, 64 minus that for odd ones).  The scalar
work sits in the first k step of a tile, in the slots behind its reads.  (The 2 x 2 tile is not limited by power; there the
scalar work, with three MFMAs to hide it behind, cost more than the lines: 2048^3 12.0 -> 12.7 us.)  Extra inputs: aw01
aw23 per-lane offsets of half 1, afix.  Registers: AW offsets of the half not due next (swapped behind every tile); s70
step of the A base (0 / 128), s96/s79 A and B request slots with ring ends s71/s72 and starts s91/s83, s76/s77 A and B read
bases of the next tile with ends s75/s74 and starts s92/s75, s73 step of the A read base, s78 temporary, s80/s81 values of
s90 at which the advance is skipped / the offsets are fixed.

CONV variants (2 x 2 and 2 x 4): the A side of a dense convolution with the im2col folded into the requests.
Tile kt is 64 channels of one filter tap (Cin % 64 == 0, at most 32 taps); a lane's chunk comes from the image at
(its pixel's byte offset at tap (0, 0)) + (tap offset, kept on the scalar unit), or, when that tap of its pixel
lies outside the image, from a constant row of theta_A bytes -- so the tile that lands in the stage is the im2col
tile itself and everything behind the request is the GEMM's loop.  Requests take a 64-bit per-lane address
(v[lo:hi], off): lo = image_lo + offset or row_lo, hi = image_hi or row_hi (the host checks that the image does
not straddle a 4 GiB line, the row table is aligned so that it cannot).  Per request: add, and, compare, two
selects.  Extra fixed registers (after VB): CT..CT+3 address temporaries (two even-aligned pairs), APIX, APIX+1
per-lane pixel offsets (request q pre-biased by -q KiB, like the table rows: the instruction offset q*1024 moves
the global address too), AMASK, AMASK+1 per-lane tap-validity bits, TABLO, TABLO+1, TABHI, IMGHI wave-uniform
address parts.  Extra SGPRs s72..s81: image_lo + tap offset, channel slice, slices per tap, kw, S, row jump
((W - S) pixels), tap bit, temporary, tap jump (pixel bytes - Cin), temporary.  Inputs apix01 amask01 (64-bit
VGPR), aptr = image, tab = row of theta_A bytes (64-bit SGPR), nc, fs (S), rowjump, tapjump (SGPR); av01 is not used.
"""
import os

def configure(tm, tn, nstage=4, conv=False, nwn=2, sets=1):
    """sets the module-level plan for TM x TN blocks of 32 x 32 per wave (2 x nwn waves per set, `sets` wave sets that
    take every sets-th k tile from stages of their own)"""
    global TM, TN, NM, A, B, RS, AV, BV, ARD0, ARD1, BRD, VA, VB, STAGE_BYTES, A_STAGE, A_DMA, N_DMA, NREAD, RSLOTS
    global AW, PAIR, B_STAGE, B_DMA, ASTEP, A_BLOCK
    global FIRST_VGPR, LAST_VGPR, NSTAGE, CT, APIX, AMASK, TABLO, TABHI, IMGHI
    assert (tm, tn) in ((4, 4), (2, 2), (2, 4)) and nstage in (3, 4)
    TM, TN, NM, NSTAGE = tm, tn, tm * tn, nstage
    # (two waves per SIMD split the register file into 128 vector and 128 accumulator registers: v127 is the last
    # one, so the convolution variants, with twelve more fixed registers, start lower)
    base = {16: 160, 4: 66 if conv else 76, 8: 50 if conv else 56}[tm * tn]
    A = [base, base + 4 * (tm + tn)]
    B = [base + 4 * tm, base + 4 * (tm + tn) + 4 * tm]
    RS = base + 8 * (tm + tn)                       # TM row-sum accumulators
    AV = RS + 4                                     # per-lane offsets of the A requests
    BV = AV + 4                                     # ... of the B requests (only the first is used: B is contiguous)
    ARD0, ARD1, BRD = BV + 4, BV + 5, BV + 6        # BRD is moved as a 64-bit pair
    VA, VB = BV + 8, BV + 9
    PAIR = tm == 4
    AW = VB + 1                                     # PAIR: the offsets of the half that is not due next
    B_STAGE = nwn * tn * 2048
    ASTEP = 64 * sets                               # bytes of a row of A from one tile of a set to its next
    FIRST_VGPR, LAST_VGPR = base, 255 if tm == 4 else VB
    CT = VB + 1 + ((VB + 1) & 1)                    # CONV: even-aligned address pairs of the two A requests
    APIX, AMASK, TABLO, TABHI, IMGHI = CT + 4, CT + 6, CT + 8, CT + 10, CT + 11
    A_STAGE = tm * 4096                             # 64 * TM rows of 64 bytes
    STAGE_BYTES = (A_STAGE + B_STAGE) * sets
    A_BLOCK = 4096 if PAIR or sets > 1 else 2048    # LDS bytes of 32 rows of A
    A_DMA, B_DMA = 2 * tm // nwn, tn                # 1 KiB requests per wave and tile: A, then B
    N_DMA = A_DMA + B_DMA
    NREAD = tm + tn                                 # LDS reads per k-step
    RSLOTS = (NREAD + 1) // 2                       # slots that carry them, two each


configure(4, 4)


def vr(base, n=4):
    return f"v[{base}:{base + n - 1}]"


class Emit:
    def __init__(self):
        self.lines = []

    def __call__(self, s):
        self.lines.append(s)

    def text(self):
        return "".join(f'    "{l}\\n"\n' for l in self.lines)


def dma(e, q):
    """one tile request: q = 0..A_DMA-1 A, then B; m0 = request stage base + slot"""
    # The instruction offset is added to the global address AND to the LDS address, so one M0 value serves the
    # four requests of a group; the per-lane A offsets come in pre-biased by -q*1024 (B is contiguous anyway).
    if q == 0:
        e("s_mov_b32 m0, s96")
        e("s_nop 0")
    if q == A_DMA and PAIR:
        e("s_mov_b32 m0, s79")
        e("s_nop 0")
    elif q == A_DMA:
        # B slots of this wave: A_STAGE further when a wave requests as many KiB of B as of A; otherwise the
        # distance is wave dependent and comes in as an operand (s85)
        e(f"s_add_u32 m0, s96, {A_STAGE}" if A_DMA == B_DMA else "s_add_u32 m0, s96, s85")
        e("s_nop 0")
    if q < A_DMA and CONV:
        lo, hi = CT + 2 * q, CT + 2 * q + 1
        e(f"v_add_u32 v{lo}, s72, v{APIX + q}")
        e(f"v_and_b32 v{hi}, s78, v{AMASK + q}")
        e(f"v_cmp_ne_u32 vcc, 0, v{hi}")
        e(f"v_cndmask_b32 v{lo}, v{TABLO + q}, v{lo}, vcc")
        e(f"v_cndmask_b32 v{hi}, v{TABHI}, v{IMGHI}, vcc")
        e(f"global_load_lds_dwordx4 v[{lo}:{hi}], off" + (f" offset:{q * 1024}" if q else ""))
    elif q < A_DMA:
        e(f"global_load_lds_dwordx4 v{AV + q}, s[86:87]" + (f" offset:{q * 1024}" if q else ""))
    else:
        e(f"global_load_lds_dwordx4 v{BV}, s[88:89]" + (f" offset:{(q - A_DMA) * 1024}" if q > A_DMA else ""))


def advance_request_pointers(e):
    if CONV:
        # next 64-channel slice; past the last slice of a tap the next tap of the filter row is (pixel bytes - Cin)
        # further (0 unless the channels are a slice of wider pixels), past the last tap of a filter row the next
        # image row (W - S) pixels further
        e("s_add_u32 s72, s72, 64")
        e("s_add_u32 s73, s73, 1")
        e("s_cmp_eq_u32 s73, s74")
        e("s_cselect_b32 s79, 1, 0")
        e("s_cselect_b32 s73, 0, s73")
        e("s_cselect_b32 s81, s80, 0")
        e("s_add_u32 s72, s72, s81")
        e("s_lshl_b32 s78, s78, s79")
        e("s_add_u32 s75, s75, s79")
        e("s_cmp_eq_u32 s75, s76")
        e("s_cselect_b32 s75, 0, s75")
        e("s_cselect_b32 s79, s77, 0")
        e("s_add_u32 s72, s72, s79")
    else:
        e(f"s_add_u32 s86, s86, {ASTEP}")
        e("s_addc_u32 s87, s87, 0")
    e("s_add_u32 s88, s88, s99")
    e("s_addc_u32 s89, s89, 0")


def pair_advance(e):
    """A request pointer to the next half; not at s90 == s80; offsets fixed at s90 == s81"""
    for q in range(A_DMA):
        e(f"v_swap_b32 v{AV + q}, v{AW + q}")
    e("s_cmp_eq_u32 s90, s80\\n s_cselect_b32 s78, 0, s70\\n s_add_u32 s86, s86, s78\\n s_addc_u32 s87, s87, 0")
    e("s_xor_b32 s70, s70, 128")
    e("s_cmp_lg_u32 s90, s81\\n s_cbranch_scc1 3f\\n " +
      "\\n ".join((f"v_add_u32 v{v + q}, %[afix], v{v + q}\\n v_subrev_u32 v{v + q}, 64, v{v + q}" if q & 1 else
                   f"v_sub_u32 v{v + q}, v{v + q}, %[afix]") for q in range(A_DMA) for v in (AV, AW)) + "\\n 3:")


def pair_advance_b(e):
    e("s_add_u32 s88, s88, s99\\n s_addc_u32 s89, s89, 0")


def ring(e, reg, step, end, start):
    """reg = reg + step, or start where that is end"""
    e(f"s_add_u32 {reg}, {reg}, {step}\\n s_cmp_eq_u32 {reg}, {end}\\n s_cselect_b32 {reg}, {start}, {reg}")


def pair_request_slots(e):
    ring(e, "s96", A_STAGE, "s71", "s91")
    ring(e, "s79", B_STAGE, "s72", "s83")


def pair_read_bases(e):
    """read bases of the next tile; the pair moves on when that is an even one"""
    ring(e, "s77", B_STAGE, "s74", "s75")
    e(f"s_xor_b32 s73, s73, {2 * A_STAGE}")
    ring(e, "s76", "s73", "s75", "s92")


def mfma(e, i, use):
    mb, nb = i // TN, i % TN
    e(f'MM("%[c{i}]", "{vr(B[use] + 4 * nb)}", "{vr(A[use] + 4 * mb)}")')


def reads(e, slot, ld, ks):
    """the two LDS reads of slot 0..RSLOTS-1: A fragments first (they are needed first), then B"""
    for j in (2 * slot, 2 * slot + 1):
        if j >= NREAD:
            continue
        if j < TM:
            e(f"ds_read_b128 {vr(A[ld] + 4 * j)}, v{VA} offset:{j * A_BLOCK}")
        else:
            nb = j - TM
            e(f"ds_read_b128 {vr(B[ld] + 4 * nb)}, v{VB} offset:{nb * 2048 + ks * 512}")


ROWSUM = True  # False: variant for weights whose zero points are all 0 (no row offsets needed)
CONV = False   # True: the A requests of a dense convolution (see the module text)


def prep_slots():
    """(first slot, slots per A fragment) of the row-sum / shift work of a k-step: the last 2*TM slots with the
    byte sums and the xor of a fragment in separate slots, or -- when the reads leave fewer -- the last TM slots
    with both in one"""
    per = 2 if NM - RSLOTS >= 2 * TM else 1
    return NM - per * TM, per


def prep(e, slot, ld):
    """fragment f = (slot - first) // per; two slots per fragment: byte sums, then xor; one slot: both"""
    first, per = prep_slots()
    f, part = (slot - first) // per, (slot - first) % per
    base = A[ld] + 4 * f
    if part == 0:
        e(f"s_waitcnt lgkmcnt({NREAD - 1 - f})")
        for c in range(4):
            if ROWSUM:
                e(f"v_sad_u8 v{RS + f}, v{base + c}, 0, v{RS + f}")
    if part == per - 1:
        for c in range(4):
            e(f"v_xor_b32 v{base + c}, s84, v{base + c}")


def step(e, use, ks_load, request, next_va, load=True, early=(), late=()):
    """TM*TN MFMAs on fragment set `use`; meanwhile fetch the next k-step's fragments into the other set
    (k-step ks_load of the stage VA/VB point at), row-sum and shift its A fragments, and optionally
    issue the tile requests.  next_va: which A offset (0/1) the NEXT step's reads use.
    PAIR: scalar work (groups that stay together) in the slots that hold neither reads nor row sums -- `early`, which the
    next read addresses need, then `late`, what is left of it behind those."""
    ld = 1 - use
    early, late = list(early), list(late)
    move_on = prep_slots()[0] - 1 if early else RSLOTS + 1
    for slot in range(NM):
        mfma(e, slot, use)
        if load and slot < RSLOTS:
            reads(e, slot, ld, ks_load)
        per = -(-N_DMA // NM)
        for q in range(slot * per, min(slot * per + per, N_DMA)):
            if request:
                dma(e, q)
        if load and slot >= prep_slots()[0]:
            prep(e, slot, ld)
        if early and slot >= RSLOTS:
            for _ in range(-(-len(early) // (move_on + 1 - slot))):
                e(early.pop(0))
        elif late and slot >= RSLOTS:
            for _ in range(-(-len(late) // (NM - slot))):
                e(late.pop(0))
        if slot == move_on and next_va is not None:
            # all reads of this step are issued: point v240/v241 at the next step's fragments
            if PAIR and next_va == 0:  # the next tile is the other one of its pair: chunk bit 2
                e(f"v_xor_b32 v{ARD0}, 64, v{ARD0}")
                e(f"v_xor_b32 v{ARD1}, 64, v{ARD1}")
            e(f"v_add_u32 v{VA}, {'s76' if PAIR else 's98'}, v{ARD0 if next_va == 0 else ARD1}")
            if next_va == 0:
                e(f"v_add_u32 v{VB}, {'s77' if PAIR else 's98'}, v{BRD}")


def wrap_stage(e, reg):
    """reg = reg mod NSTAGE for reg in 0..NSTAGE"""
    if NSTAGE == 4:
        e(f"s_and_b32 {reg}, {reg}, 3")
    else:
        e(f"s_cmp_eq_u32 {reg}, {NSTAGE}")
        e(f"s_cselect_b32 {reg}, 0, {reg}")


def stage_offset(e, dst, src):
    """dst = src * STAGE_BYTES"""
    if STAGE_BYTES & (STAGE_BYTES - 1) == 0:
        e(f"s_lshl_b32 {dst}, {src}, {STAGE_BYTES.bit_length() - 1}")
    else:
        e(f"s_mul_i32 {dst}, {src}, {STAGE_BYTES}")


def rotate_stage(e):
    """end of a tile: stage index += 1 (mod NSTAGE); recompute the read bases"""
    e("s_add_u32 s93, s93, 1")
    wrap_stage(e, "s93")
    e("s_mov_b32 s97, s98")
    e("s_add_u32 s94, s93, 1")
    wrap_stage(e, "s94")
    stage_offset(e, "s94", "s94")
    e("s_add_u32 s98, s92, s94")


def tile(e, wait_vm, request, last=False):
    if PAIR:
        tile_pair(e, wait_vm, request, last)
        return
    # k-step 0 of tile t: consume set 0, fetch (t, 1) into set 1 from the current stage
    step(e, use=0, ks_load=1, request=False, next_va=None if last else 0)
    if last:
        e("s_waitcnt lgkmcnt(0)")
        step(e, use=1, ks_load=0, request=False, next_va=None, load=False)
        return
    # every wave: its requests for tile t+1 have landed, its reads of tile t are done
    e(f"s_waitcnt vmcnt({wait_vm}) lgkmcnt(0)")
    e("s_barrier")
    if request:
        stage_offset(e, "s94", "s93")
        e("s_add_u32 s96, s91, s94")
    # k-step 1 of tile t: consume set 1, fetch (t+1, 0) into set 0 from the next stage
    step(e, use=1, ks_load=0, request=request, next_va=1)
    if request:
        advance_request_pointers(e)
    rotate_stage(e)
    e("s_waitcnt lgkmcnt(0)")


def tile_pair(e, wait_vm, request, last):
    """tile() of the PAIR loops: the same steps and waits; the pointers are moved on in the first k step, behind its reads"""
    early, late = Emit(), Emit()
    if not last:
        pair_read_bases(early)
    if request:
        pair_advance(late)
        pair_advance_b(late)
        pair_request_slots(late)
    step(e, use=0, ks_load=1, request=False, next_va=None if last else 0, early=early.lines, late=late.lines)
    if last:
        e("s_waitcnt lgkmcnt(0)")
        step(e, use=1, ks_load=0, request=False, next_va=None, load=False)
        return
    e(f"s_waitcnt vmcnt({wait_vm}) lgkmcnt(0)")
    e("s_barrier")
    step(e, use=1, ks_load=0, request=request, next_va=1)
    e("s_waitcnt lgkmcnt(0)")


def generate_loop(rowsum, conv=False):
    global ROWSUM, CONV
    ROWSUM, CONV = rowsum, conv
    assert not conv or TM == 2
    e = Emit()
    # ---- unpack operands into the fixed registers
    if conv:
        e(f"v_mov_b64 v[{APIX}:{APIX + 1}], %[apix01]")
        e(f"v_mov_b64 v[{AMASK}:{AMASK + 1}], %[amask01]")
        e("s_mov_b64 s[72:73], %[tab]")
        e(f"v_mov_b32 v{TABLO}, s72")
        e("s_sub_u32 s72, s72, 1024")
        e(f"v_mov_b32 v{TABLO + 1}, s72")
        e(f"v_mov_b32 v{TABHI}, s73")
        e("s_mov_b64 s[72:73], %[aptr]")
        e(f"v_mov_b32 v{IMGHI}, s73")
        e("s_mov_b32 s73, 0")
        e("s_mov_b32 s74, %[nc]")
        e("s_mov_b32 s75, 0")
        e("s_mov_b32 s76, %[fs]")
        e("s_mov_b32 s77, %[rowjump]")
        e("s_mov_b32 s78, 1")
        e("s_mov_b32 s80, %[tapjump]")
    else:
        e(f"v_mov_b64 v[{AV}:{AV + 1}], %[av01]")
    if A_DMA == 4:
        e(f"v_mov_b64 v[{AV + 2}:{AV + 3}], %[av23]")
    if PAIR:
        e(f"v_mov_b64 v[{AW}:{AW + 1}], %[aw01]")
        if TM == 4:
            e(f"v_mov_b64 v[{AW + 2}:{AW + 3}], %[aw23]")
    e(f"v_mov_b64 v[{BV}:{BV + 1}], %[bv01]")
    if TM == 4:
        e(f"v_mov_b64 v[{BV + 2}:{BV + 3}], %[bv23]")
    e(f"v_mov_b64 v[{ARD0}:{ARD1}], %[ard]")
    e(f"v_mov_b64 v[{BRD}:{BRD + 1}], %[brd]")
    e("s_mov_b32 s84, 0x80808080")
    if A_DMA != B_DMA:
        e("s_mov_b32 s85, %[bofs]")
    if not conv:
        e("s_mov_b64 s[86:87], %[aptr]")
    e("s_mov_b64 s[88:89], %[bptr]")
    e(f"s_sub_u32 s90, %[kt], {NSTAGE}")
    e("s_mov_b32 s91, %[ldsdma]")
    e("s_mov_b32 s92, %[lds]")
    e("s_mov_b32 s99, %[bstep]")
    for f in range(TM):
        e(f"v_mov_b32 v{RS + f}, 0")
    # The first NSTAGE tiles (PAIR: five halves of A, four tiles of B) have been requested by the surrounding C++ code, in
    # the order of the loop; the pointers come in at the next tile (PAIR: at the last requests, advanced in the first tile).
    # The convolution requests them here.
    if PAIR:
        e("s_mov_b32 s70, 0")
        e(f"s_add_u32 s96, s91, {4 * A_STAGE}")
        e(f"s_add_u32 s79, s91, {6 * A_STAGE + 3 * B_STAGE}")
        # an even number of tiles: skip the advance in the last tile that requests (s90 == 1); an odd one: fix the offsets
        # in the one before, in front of the requests for the last pair (s90 == 2)
        e("s_and_b32 s78, s90, 1")
        e("s_cmp_eq_u32 s78, 0\\n s_cselect_b32 s80, 1, -1\\n s_cselect_b32 s81, -1, 2")
        e(f"s_add_u32 s71, s91, {6 * A_STAGE}")
        e("s_mov_b32 s83, s71")
        e(f"s_add_u32 s72, s83, {4 * B_STAGE}")
        e(f"s_mov_b32 s73, {2 * A_STAGE}")
        e(f"s_add_u32 s75, s92, {6 * A_STAGE}")
        e(f"s_add_u32 s74, s75, {4 * B_STAGE}")
        e("s_mov_b32 s76, s92")
        e("s_mov_b32 s77, s75")
        e("s_mov_b32 s97, s92")
    else:
        for st in range(NSTAGE if conv else 0):
            e(f"s_add_u32 s96, s91, {st * STAGE_BYTES}")
            for q in range(N_DMA):
                dma(e, q)
            advance_request_pointers(e)
        e(f"s_add_u32 s98, s92, {STAGE_BYTES}")
        e("s_mov_b32 s93, 0")
        e("s_mov_b32 s97, s92")
    e(f"s_waitcnt vmcnt({(NSTAGE - 1) * N_DMA})")
    e("s_barrier")
    # ---- fragments (0, 0) into set 0
    e(f"v_add_u32 v{VA}, s97, v{ARD0}")
    e(f"v_add_u32 v{VB}, s97, v{BRD}")
    if PAIR:
        e(f"v_add_u32 v{VB}, {6 * A_STAGE}, v{VB}")
    for slot in range(RSLOTS):
        reads(e, slot, 0, 0)
    for f in range(TM):
        e(f"s_waitcnt lgkmcnt({NREAD - 1 - f})")
        for c in range(4):
            if ROWSUM:
                e(f"v_sad_u8 v{RS + f}, v{A[0] + 4 * f + c}, 0, v{RS + f}")
        for c in range(4):
            e(f"v_xor_b32 v{A[0] + 4 * f + c}, s84, v{A[0] + 4 * f + c}")
    e("s_waitcnt lgkmcnt(0)")
    e(f"v_add_u32 v{VA}, s97, v{ARD1}")
    e("s_nop 1")
    # ---- steady state: KT-NSTAGE tiles, each requesting tile t+NSTAGE
    e("s_cmp_eq_u32 s90, 0")
    e("s_cbranch_scc1 2f")
    e("1:")
    tile(e, (NSTAGE - 2) * N_DMA, request=True)
    e("s_sub_u32 s90, s90, 1")
    e("s_cmp_lg_u32 s90, 0")
    e("s_cbranch_scc1 1b")
    e("2:")
    # ---- drain: nothing left to request; the tiles still in flight are fewer with every tile
    for younger in range(NSTAGE - 2, -1, -1):
        tile(e, younger * N_DMA, request=False)
    tile(e, 0, request=False, last=True)
    # ---- results: let the last MFMAs retire, hand the row sums back
    e("s_nop 15")
    e("s_nop 15")
    e("s_nop 15")
    e(f"v_mov_b64 %[rs01], v[{RS}:{RS + 1}]")
    if TM == 4:
        e(f"v_mov_b64 %[rs23], v[{RS + 2}:{RS + 3}]")
    return e.lines


def macro(name, lines):
    """the loop as a macro of MM, which writes one MFMA (accumulator, B fragment, A fragment): the caller chooses which of the
    two comes first, and so whether a lane ends up with columns of one row or rows of one column"""
    return f"#define {name}(MM) \\\n" + "".join(f"  {l} \\\n" if l.startswith("MM(") else f'  "{l}\\n" \\\n' for l in lines) + "  \"\"\n"


def generate():
    out = "// GENERATED by gen_tile_loop.py -- do not edit.\n"
    for tm, tn, nstage, suffix in ((4, 4, 4, ""), (2, 2, 4, "_2X2"), (2, 4, 3, "_2X4")):
        configure(tm, tn, nstage)
        clob = [f'"v{i}"' for i in range(FIRST_VGPR, LAST_VGPR + 1)] + [f'"s{i}"' for i in range(70 if PAIR else 84, 100)] + \
               ['"scc"', '"memory"']
        for name, rowsum in (("QG_TILE_LOOP_ASM", True), ("QG_TILE_LOOP_ASM_NOROWSUM", False)):
            out += macro(name + suffix, generate_loop(rowsum))
        out += f"#define QG_TILE_LOOP_CLOBBERS{suffix} " + ", ".join(clob) + "\n"
        if tm == 2:
            configure(tm, tn, nstage, conv=True)
            clob = [f'"v{i}"' for i in range(FIRST_VGPR, IMGHI + 1)] + [f'"s{i}"' for i in range(72, 82)] + \
                   [f'"s{i}"' for i in range(84, 100)] + ['"vcc"', '"scc"', '"memory"']
            for name, rowsum in (("QG_TILE_LOOP_ASM_CONV", True), ("QG_TILE_LOOP_ASM_CONV_NOROWSUM", False)):
                out += macro(name + suffix, generate_loop(rowsum, conv=True))
            out += f"#define QG_TILE_LOOP_CLOBBERS_CONV{suffix} " + ", ".join(clob) + "\n"
    # the 128 x 64 tile: 64 x 64 per wave, four sets of two waves
    configure(2, 2, 3, nwn=1, sets=4)
    clob = [f'"v{i}"' for i in range(FIRST_VGPR, LAST_VGPR + 1)] + [f'"s{i}"' for i in range(84, 100)] + ['"scc"', '"memory"']
    for name, rowsum in (("QG_TILE_LOOP_ASM_2X2K4", True), ("QG_TILE_LOOP_ASM_NOROWSUM_2X2K4", False)):
        out += macro(name, generate_loop(rowsum))
    out += "#define QG_TILE_LOOP_CLOBBERS_2X2K4 " + ", ".join(clob) + "\n"
    configure(4, 4)
    return out


if __name__ == "__main__":
    here = os.path.dirname(os.path.abspath(__file__))
    with open(os.path.join(here, "tile_loop_asm.inc"), "w") as f:
        f.write(generate())
    print("wrote tile_loop_asm.inc")
