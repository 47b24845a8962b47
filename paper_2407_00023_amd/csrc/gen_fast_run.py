#!/usr/bin/env python3
"""Writes fast_run.inc: the tiles of the bf16 extend-attention kernel as gfx950 assembly.

One inline-assembly statement per kernel instance holds every kind of tile, for head dimension 128 or 64 and 32 packed query
rows per wave, with every register chosen here.  (Left to the compiler's register allocator the 64 output accumulators
are split around the phases of a tile and copied every tile, and spill reloads inside the loop serialise the
global -> LDS loads behind them; and several statements, each with its fixed registers, made the compiler spill
everything it held around them.)  A mode operand picks the kind: runs of consecutive unmasked tiles that issue the
next tile's loads themselves (its rows in the pool through slot ids, 32-bit or 64-bit addresses, as codes of the fp8
pool, or in the extend tokens), and single tiles, plain or with keys hidden from rows, whose loads the caller issues.

The products are 16x16x32 MFMAs: what bounds the large launches is the chip's power, and these take less of it than 32x32x16 ones
for the same work (loops of nothing else, operands with busy bits, all of the chip, TFLOP/s: 2,205 to 2,260 against 1,905 to 1,940 on one
box, 1,880 to 2,130 against 1,640 to 1,810 on another).  A lane then holds two query rows (l % 16 and 16 more) and, of a block of 32 keys, 4 (l / 16) .. + 3 of
each half.

A tile is 64 MFMAs (32 at head dimension 64), in four phases of NB fragments, each multiplied with the rows 0..15 first and,
when all have been, with the rows 16..31; what stands behind an MFMA in the stream runs in its shadow:
    S0 = K(block 0) Q^T  | addresses + issue of the next tile's global -> LDS loads; slot ids of the tile after next
    S1 = K(block 1) Q^T  | probabilities 2^(c S0 - m) from the second half of S0 on, their sums
    (leave with status 1 if a row's sum exceeds the limit: block 0 outgrew the running maximum m)
    O += V(block 0) P0   | probabilities 2^(c S1 - m), their sums
    (leave with status 2)
    O += V(block 1) P1   | half-way: wait for this wave's loads, workgroup barrier
A fragment buffer is free once the rows 16..31 have been multiplied and takes the fragment of the next phase with its number, eight
MFMAs ahead of its use; the barrier stands behind the last read of this tile, so that the next tile's first fragments are read in
the shadow of this tile's last products.  (fp8 pool: the rows that landed are turned into bfloat16 behind the last product, and the
barrier follows.)

An MFMA takes 16 cycles of the matrix pipe and, of the port that it shares with the vector instructions, two of their slots of
four cycles (an exponential two as well): two vector instructions behind every MFMA are free, each one more costs four cycles.  So
the schedule is written for few of them, spread evenly: a row's place is worked out by one lane and broadcast to the others that
fetch it, row sums are products with ones (dot products wait for the matrix pipe to run dry, and the pipe for them).
LDS reads are awaited two fragments at a time by counting them (they return in order).  Wait states the hardware does not
interlock are written out, other work standing in them where there is any: an MFMA and an ALU read of its result (eight slots of four
cycles), a transcendental and a use of its result (one instruction), a write of M0 and the load that uses it (one), a
vector write of a register and a broadcast from it (two), a comparison and a selection by it (two); check_waits() holds the tiles to them.
The loop is written out for both ring slots, so that every LDS offset is an immediate and no address register changes
between tiles.

Measured, the loop alone with rows from the L2s, all of the chip, per 256 rows and 64 keys on a compute unit: phases of 32x32x16 MFMAs
with dot products 1.77 us (3,090 cycles at 1,740 MHz); 16x16x32, each fragment with all rows at once and the probabilities in two of
four phases 1.65 (3,130 at 1,900); this order 1.60 (2,970 at 1,860).

Run:  python gen_fast_run.py  (the build does)."""
import os
import re


def shape(D):
    """Sizes and vector registers for one head dimension.  D = 128 fills 256 registers (two waves on a SIMD), D = 64 keeps to
    168 (three): half the arithmetic per tile, so more of the time goes to the exponentials of the wave itself, and a third
    wave fills it."""
    global KS, NB, ROWB, TILEB, STAGEB, UPW, RPB, NFR
    global ACC, Q, SC0, SC1, PB0, PB1, FR, ONE, KRD, VRD, SLN, L, NEGM, KOFF0, VOFF0, ROWI, KRD0, VRD0, T, ROWOFF, SWZ, LIM, NEGINF, FIRST_V
    KS, NB = D // 32, D // 16           # k-slices of QK^T, head-dim blocks of O^T
    ROWB, TILEB, STAGEB = 2 * D, 128 * D, 256 * D
    UPW, RPB = D // 32, 512 // D        # 1 KB load blocks per wave and tensor, rows per block
    NFR = NB                            # fragment buffers: those of a phase
    # everything from FIRST_V up belongs to the assembly
    top = 256 if D == 128 else 168

    def take(n):
        nonlocal top
        top -= n
        return top
    ACC = [[take(4) for _ in range(NB)][::-1] for _ in range(2)]    # [rows 0..15 / 16..31 of the wave][head-dim block]
    Q = [[take(4) for _ in range(KS)][::-1] for _ in range(2)]      # [row block][k-slice]
    SC0, SC1 = take(16), take(16)       # scores: register 4 (2 key half + row block) + i
    PB0, PB1 = take(8), take(8)         # probabilities: 4 x row block + 2 x key half + i / 2
    FR = [take(4) for _ in range(NFR)][::-1]
    ONE = take(4)                       # the A operand that sums rows
    KRD = [take(1) for _ in range(KS)][::-1]
    VRD = [take(1) for _ in range(NB)][::-1]
    SLN = [take(1) for _ in range(1 if D == 128 else UPW)][::-1]
    L = [take(1) for _ in range(2)]
    NEGM = [take(1) for _ in range(2)]
    KOFF0, VOFF0, ROWI, KRD0, VRD0 = [take(1) for _ in range(5)]
    if (top - 7) % 2:
        take(1)                         # (pairs of T hold 64-bit addresses)
    T = [take(1) for _ in range(7)][::-1]
    ROWOFF = [take(1) for _ in range(2)]
    if D == 128:
        SWZ = [take(1) for _ in range(2)]
    LIM, NEGINF = T[0:2], T[6]          # masked single tiles (they issue no loads: the T registers are free)
    FIRST_V = top


MASKS = [72, 74]                        # two scalar register pairs for the comparisons of masked single tiles
# ---- scalar registers ----
P0, RING, STATUS, PEND = 40, 41, 42, 43
SLOTS, BASE_K, BASE_V = 44, 46, 48     # 64-bit pairs: slot ids; K rows (pool or k_ext); V rows (pool + K->V distance, or v_ext)
C = 52                                  # s[52:59]: see the operand list in emit()
C2 = 60                                 # s[60:63]
S_T = [68, 69, 70, 71]                  # scratch scalars
C_SHIFT, C_MASK, C_PSTRIDE, C_NSLOT1, C_P1, C_XSTRIDE, C_EXTMAX, C_LDSW = range(C, C + 8)
C_128, C_192, C_P, C_SCALE = range(C2, C2 + 4)
# the fp8 pool's runs (kind pool8) take other values in four of the operands, and one operand more:
C_EXPPAGE, C_EXPV = C_XSTRIDE, C_EXTMAX   # bytes from one page's row exponents to the next page's; from a K row's exponent to its V row's
EXP_BASE = C_128                          # s[60:61]: the row exponents of this KV head
EXST = 51                                 # LDS address of this wave's staging area for row exponents
LIMIT = "0x53800000"   # 2^40: a row's probabilities of one key block may sum to this much before the run is left
ONES = "0x3f803f80"    # bf16 (1, 1)


def v(i, n=1):
    return f"v{i}" if n == 1 else f"v[{i}:{i + n - 1}]"


def s(i, n=1):
    return f"s{i}" if n == 1 else f"s[{i}:{i + n - 1}]"


def v_swizzle(u):
    """Load block u of a wave holds rows 4 u + lane / 16 (heads of 64: 8 u + lane / 8) of its share: what the swizzle of their V
    rows differs by from that of block 0, in bytes."""
    return 16 * (2 * (u & 1) + (u >> 1)) if ROWB == 256 else 16 * u


class Stream:
    def __init__(self):
        self.lines = []
        self.lds = []      # ids of LDS reads in flight, oldest first
        self.next_id = 0

    def emit(self, text):
        self.lines.append(text)

    def lds_read(self, text):
        self.emit(text)
        self.lds.append(self.next_id)
        self.next_id += 1
        return self.next_id - 1

    def wait_lds(self, op_id):
        """Wait until LDS read op_id (and every older one) has returned."""
        if op_id not in self.lds:
            return
        after = len(self.lds) - 1 - self.lds.index(op_id)
        self.emit(f"s_waitcnt lgkmcnt({after})")
        self.lds = self.lds[len(self.lds) - after:] if after else []


def tile(st, kind, ring, upw):
    """One tile that sits in ring slot `ring`; the next tile is loaded into the other slot.  st.lds: the reads of its first
    fragments, under way already (not for the kinds in st.no_prefetch)."""
    e = st.emit
    idle = kind.endswith("_idle")
    name = kind[:-5] if idle else kind
    ext, wide, raw8 = name == "ext", name == "pool64", name == "pool8"
    noload, masked = kind in ("plain", "masked"), kind == "masked"   # (single tiles: the kernel issues the next tile's loads itself)
    here, there = ring * STAGEB, (ring ^ 1) * STAGEB
    NF = NB       # K fragments of a key block (two halves of 16 keys x KS slices), and its V^T fragments (one per head-dim block)
    NK = 2 * NF   # ... of a tile
    last = dict(enumerate(st.lds))   # fragment number (0 .. NK - 1 K, NK .. V) -> id of its last LDS read
    assert len(last) == (0 if kind in st.no_prefetch else NF)

    def read_frag(f, slot=here):
        buf = FR[f % NFR]
        if f < NK:   # K fragment: key block, k-slice, half of the block's keys
            blk, x = divmod(f, NF)
            sl, kb = divmod(x, 2)
            off = slot + blk * 32 * ROWB + kb * 16 * ROWB
            o = f" offset:{off}" if off else ""
            return st.lds_read(f"ds_read_b128 {v(buf, 4)}, {v(KRD[sl])}{o}")
        # V^T fragment: key block, head-dim block; its two halves are 16 keys apart
        blk, b = divmod(f - NK, NF)
        off = slot + blk * 32 * ROWB
        o = f" offset:{off}" if off else ""
        st.lds_read(f"ds_read_b64_tr_b16 {v(buf, 2)}, {v(VRD[b])}{o}")
        return st.lds_read(f"ds_read_b64_tr_b16 {v(buf + 2, 2)}, {v(VRD[b])} offset:{off + 16 * ROWB}")

    def mfma(dst, a, b, c):
        e(f"v_mfma_f32_16x16x32_bf16 {dst}, {a}, {b}, {c}")

    def newbcast(u):
        return f"row_newbcast:{u} row_mask:0xf bank_mask:0xf"

    def load_base():
        """Heads of 128: where the next tile's rows lie.  Lane 16 j + u (and the others with the same l % 4 = u) holds the slot of
        row 4 u + j of the wave's sixteen, the row that the lanes 16 j .. 16 j + 15 fetch in load block u, and works out its place
        once; load_piece() takes it from there by a broadcast inside the sixteen.  (Worked out by every lane for its four rows, this
        was 29 vector instructions and four loads of slot ids per tile; now 16 and one.)  ROWOFF: byte offsets of the rows from
        the bases, for K and V, with what the swizzle of block u differs by from block 0's already in them (rows are aligned to
        256 bytes, so nothing carries).  Two instructions have to stand between these results and a broadcast of them."""
        k, w = ROWOFF
        if ext:
            # position of the row in the extend tokens, clamped to the last valid key; times the token stride
            x = [f"s_add_u32 {s(S_T[2])}, {s(P0)}, 64", f"s_sub_u32 {s(S_T[2])}, {s(S_T[2])}, {s(C_P)}", f"v_add_u32 {v(T[0])}, {s(S_T[2])}, {v(ROWI)}",
                 f"v_min_i32 {v(T[0])}, {s(C_EXTMAX)}, {v(T[0])}", f"v_mul_u32_u24 {v(T[0])}, {s(C_XSTRIDE)}, {v(T[0])}"]
        else:
            # slot id (never outside the pool) -> page, offset in the page
            x = [f"v_med3_i32 {v(T[0])}, {v(SLN[0])}, 0, {s(C_NSLOT1)}", f"v_lshrrev_b32 {v(T[1])}, {s(C_SHIFT)}, {v(T[0])}",
                 f"v_and_b32 {v(T[0])}, {s(C_MASK)}, {v(T[0])}"]
            if wide:
                # number of the K row from the head's first, in rows of 256 bytes, then in units of 16 bytes (the 64-bit shift-and-add
                # shifts by 4 at most; below 2^32 for pools of up to 64 GB)
                return x + [f"v_mad_u32_u24 {v(T[0])}, {v(T[1])}, {s(C_PSTRIDE)}, {v(T[0])}", f"v_lshlrev_b32 {v(k)}, 4, {v(T[0])}",
                            f"v_mov_b32 {v(T[1])}, 0", "s_nop 0"]
            if raw8:
                # ROWOFF: of the row's codes, and of its K exponent
                return x + [f"v_mad_u32_u24 {v(w)}, {v(T[1])}, {s(C_EXPPAGE)}, {v(T[0])}", f"v_lshlrev_b32 {v(T[0])}, 7, {v(T[0])}",
                            f"v_mad_u32_u24 {v(k)}, {v(T[1])}, {s(C_PSTRIDE)}, {v(T[0])}", f"v_add_u32 {v(T[3])}, {s(C_EXPV)}, {v(w)}", "s_nop 0"]
            # ... -> byte offset of the K row
            x += [f"v_lshlrev_b32 {v(T[0])}, 8, {v(T[0])}", f"v_mad_u32_u24 {v(T[0])}, {v(T[1])}, {s(C_PSTRIDE)}, {v(T[0])}"]
        return x + [f"v_xor_b32 {v(k)}, {v(SWZ[0])}, {v(T[0])}", f"v_xor_b32 {v(w)}, {v(SWZ[1])}, {v(T[0])}", "s_nop 0"]

    def load_piece(u, which):
        """The load of block u of the next tile's K rows, or of its V rows.  (M0 first: the address arithmetic that follows is the
        wait state the load needs after it.)"""
        m0 = there + u * 1024 + (TILEB if which else 0)
        x = [f"s_add_u32 m0, {s(C_LDSW)}, {m0}" if m0 else f"s_mov_b32 m0, {s(C_LDSW)}"]
        base, off0 = (BASE_V, VOFF0) if which else (BASE_K, KOFF0)
        if wide:
            # (T[0], T[1]) = (row number in units of 16 bytes, 0), the 64-bit operand; the bases are 256-byte aligned: adding the
            # offset inside the row never carries
            if which == 0:
                x.append(f"v_mov_b32_dpp {v(T[0])}, {v(ROWOFF[0])} {newbcast(u)}")
            to = T[4] if which else T[2]
            swz = v_swizzle(u) if which else [0, 64, s(C_128), s(C_192)][u]
            return x + [f"v_lshl_add_u64 {v(to, 2)}, {v(T[0], 2)}, 4, {s(base, 2)}", f"v_xad_u32 {v(to)}, {v(off0)}, {swz}, {v(to)}",
                        f"global_load_lds_dwordx4 {v(to, 2)}, off"]
        if ROWB == 256:
            x.append(f"v_xor_b32_dpp {v(T[2 + which])}, {v(ROWOFF[which])}, {v(off0)} {newbcast(u)}")
        else:
            if which == 0 and ext:
                # position of the row in the extend tokens, clamped to the last valid key; times the token stride
                x += [f"s_add_u32 {s(S_T[2])}, {s(P0)}, {64 + RPB * u}", f"s_sub_u32 {s(S_T[2])}, {s(S_T[2])}, {s(C_P)}",
                      f"v_add_u32 {v(T[0])}, {s(S_T[2])}, {v(ROWI)}", f"v_min_i32 {v(T[0])}, {s(C_EXTMAX)}, {v(T[0])}",
                      f"v_mul_u32_u24 {v(ROWOFF[0])}, {s(C_XSTRIDE)}, {v(T[0])}"]
            elif which == 0:
                # slot id (never outside the pool) -> page, offset in the page -> byte offset of the K row
                x += [f"v_med3_i32 {v(T[0])}, {v(SLN[u])}, 0, {s(C_NSLOT1)}", f"v_lshrrev_b32 {v(T[1])}, {s(C_SHIFT)}, {v(T[0])}",
                      f"v_and_b32 {v(T[0])}, {s(C_MASK)}, {v(T[0])}", f"v_lshlrev_b32 {v(T[0])}, {ROWB.bit_length() - 1}, {v(T[0])}",
                      f"v_mad_u32_u24 {v(ROWOFF[0])}, {v(T[1])}, {s(C_PSTRIDE)}, {v(T[0])}"]
            x.append(f"v_xad_u32 {v(T[2 + which])}, {v(off0)}, {v_swizzle(u) if which else 64 * u}, {v(ROWOFF[0])}")
        return x + [f"global_load_lds_dwordx4 {v(T[2 + which])}, {s(base, 2)}"]

    def load_piece8(u, which):
        """fp8 pool: block u of the next tile's K or V rows as codes.  A row's 128 codes go to the first half of the 256 LDS bytes its
        bfloat16 form will take (the lanes that would fetch the second half are switched off).  T[6] = 16 (lane % 16)."""
        x = [f"s_add_u32 m0, {s(C_LDSW)}, {there + u * 1024 + (TILEB if which else 0)}"]
        if which == 0:
            x.append(f"v_add_u32_dpp {v(T[2])}, {v(ROWOFF[0])}, {v(T[6])} {newbcast(u)}")
        return x + [f"s_mov_b64 exec, {s(MASKS[0], 2)}", f"global_load_lds_dwordx4 {v(T[2])}, {s(BASE_V if which else BASE_K, 2)}", "s_mov_b64 exec, -1"]

    def load_exponents():
        """... and the exponents of the wave's sixteen K and sixteen V rows, one byte each, to its staging area: lane 16 j + u fetches
        those of row 4 u + j."""
        return [f"s_mov_b32 m0, {s(EXST)}", f"s_mov_b64 exec, {s(MASKS[1], 2)}", f"global_load_lds_ubyte {v(ROWOFF[1])}, {s(EXP_BASE, 2)}",
                f"s_add_u32 m0, {s(EXST)}, 256", "s_nop 0", f"global_load_lds_ubyte {v(T[3])}, {s(EXP_BASE, 2)}", "s_mov_b64 exec, -1"]

    def decode8():
        """fp8 pool, after this wave's loads have landed: its rows of the next tile from codes to bfloat16, in place.
        All sixteen lanes of a row read their 8 codes before any of them writes, and nobody else touches the row
        before the barrier.  The fragment and score registers are free here."""
        DEC_RAW, DEC_EXP, DEC_OUT = FR[0], FR[4], SC1   # codes (16 registers), exponents (8), bfloat16 (32)
        e(f"v_and_b32 {v(T[0])}, 3, {v(ROWI)}")                           # lane / 16
        e(f"v_lshl_add_u32 {v(T[1])}, {v(T[0])}, 8, {s(C_LDSW)}")          # this lane's row in load block 0, ring slot 0
        e(f"v_lshl_add_u32 {v(T[5])}, {v(T[0])}, 6, {s(EXST)}")            # the words that hold its rows' exponents
        e(f"v_lshlrev_b32 {v(T[0])}, 4, {v(T[0])}")
        e(f"v_xor_b32 {v(T[6])}, {v(KOFF0)}, {v(T[0])}")                   # 16 (lane % 16)
        e(f"v_add_u32 {v(T[6])}, {v(T[1])}, {v(T[6])}")                    # where this lane's 16 bytes of a load block go
        e(f"v_lshrrev_b32 {v(T[2])}, 1, {v(KOFF0)}")
        e(f"v_lshrrev_b32 {v(T[3])}, 1, {v(VOFF0)}")
        for u in range(upw):
            if 32 * u <= 64:
                e(f"v_xad_u32 {v(T[4])}, {v(T[2])}, {32 * u}, {v(T[1])}")
            else:   # (not an inline constant)
                e(f"v_xor_b32 {v(T[4])}, {32 * u}, {v(T[2])}")
                e(f"v_add_u32 {v(T[4])}, {v(T[1])}, {v(T[4])}")
            st.lds_read(f"ds_read_b64 {v(DEC_RAW + 4 * u, 2)}, {v(T[4])} offset:{there + u * 1024}")
            e(f"v_xad_u32 {v(T[4])}, {v(T[3])}, {v_swizzle(u) // 2}, {v(T[1])}")
            st.lds_read(f"ds_read_b64 {v(DEC_RAW + 4 * u + 2, 2)}, {v(T[4])} offset:{there + TILEB + u * 1024}")
        st.lds_read(f"ds_read_b128 {v(DEC_EXP, 4)}, {v(T[5])}")
        st.lds_read(f"ds_read_b128 {v(DEC_EXP + 4, 4)}, {v(T[5])} offset:256")
        for u in range(upw):
            for t in range(2):
                if u == 0 and t == 0:
                    e("s_waitcnt lgkmcnt(0)")
                    st.lds.clear()
                ex, raw, out = DEC_EXP + 4 * t + u, DEC_RAW + 4 * u + 2 * t, DEC_OUT + 4 * (2 * u + t)
                e(f"v_bfe_i32 {v(ex)}, {v(ex)}, 0, 8")
                e(f"v_lshl_add_u32 {v(ex)}, {v(ex)}, 23, 0x3f800000")       # 2^k as a float
                for h in range(2):
                    e(f"v_cvt_scalef32_pk_bf16_fp8 {v(out + 2 * h)}, {v(raw + h)}, {v(ex)}")
                    e(f"v_cvt_scalef32_pk_bf16_fp8 {v(out + 2 * h + 1)}, {v(raw + h)}, {v(ex)} op_sel:[1,0,0]")
                e(f"ds_write_b128 {v(T[6])}, {v(out, 4)} offset:{there + t * TILEB + u * 1024}")
        e("s_waitcnt lgkmcnt(0)")

    late = []      # probability pairs whose conversion is still to come: [(register, exponential, exponential)]

    def convert():
        """Conversion of the oldest pair of exponentials (never the instruction after them: a transcendental and the use
        of its result want one other instruction between them)."""
        pb, t0, t1 = late.pop(0)
        return f"v_cvt_pk_bf16_f32 {v(pb)}, {v(t0)}, {v(t1)}"

    def exp_piece(sc, pb, idx):
        """Two probabilities of a score block: row block idx / 4, registers 2 h, 2 h + 1 of key half kb; the conversion of the
        piece before stands behind their exponentials (two pairs of registers in turn).  Masked tiles: register i of a lane
        holds the key at offset 16 kb + i from the lane's first key of the block, visible if that is below the lane's limit;
        the exponent of a hidden key becomes -inf (two comparisons ahead of the two selections, so that their results
        have reached the scalar registers)."""
        rb, (kb, h) = idx // 4, divmod(idx % 4, 2)
        at = sc + 4 * (2 * kb + rb) + 2 * h
        t0, t1 = (T[4], T[5]) if idx % 2 == 0 else (T[2], T[3])
        x = []
        if masked:
            for k in range(2):
                x.append(f"v_cmp_gt_i32 {s(MASKS[k], 2)}, {v(LIM[rb])}, {16 * kb + 2 * h + k}")
        x.append(f"v_fma_f32 {v(t0)}, {v(at)}, {s(C_SCALE)}, {v(NEGM[rb])}")
        x.append(f"v_fma_f32 {v(t1)}, {v(at + 1)}, {s(C_SCALE)}, {v(NEGM[rb])}")
        if masked:
            x.append(f"v_cndmask_b32 {v(t0)}, {v(NEGINF)}, {v(t0)}, {s(MASKS[0], 2)}")
            x.append(f"v_cndmask_b32 {v(t1)}, {v(NEGINF)}, {v(t1)}, {s(MASKS[1], 2)}")
        x.append(f"v_exp_f32 {v(t0)}, {v(t0)}")
        x.append(f"v_exp_f32 {v(t1)}, {v(t1)}")
        late.append((pb + 4 * rb + 2 * kb + h, t0, t1))
        if len(late) > 1:
            x.append(convert())
        return x

    def sum_products(sc, pb):
        """The row sums of a key block, as a product with ones.  (The block's scores are not needed any more.)"""
        for rb in range(2):
            mfma(v(sc + 4 * rb, 4), v(ONE, 4), v(pb + 4 * rb, 4), "0")

    def check_sums(sc, over):
        e("s_nop 2")
        e(f"v_max_u32 {v(ROWOFF[0])}, {v(sc)}, {v(sc + 4)}")
        e(f"v_cmp_lt_u32 vcc, {LIMIT}, {v(ROWOFF[0])}")
        e(f"s_cbranch_vccnz {over}{st.kind_end}")
        for rb in range(2):
            e(f"v_add_f32 {v(L[rb])}, {v(L[rb])}, {v(sc + 4 * rb)}")

    def end_of_tile():
        e(f"s_add_u32 {s(P0)}, {s(P0)}, 64")
        e(f"s_mov_b32 {s(RING)}, {ring ^ 1}")
        e(f"s_cmp_lt_i32 {s(P0)}, {s(PEND)}")

    def slot_ids():
        """Slot ids of this lane's rows (heads of 128: of its one row, see load_base) in the tile after the next one; rows outside the
        prefix repeat the last prefix slot."""
        x = []
        for u in range(len(SLN)):
            x += [f"s_add_u32 {s(S_T[3])}, {s(P0)}, {128 + RPB * u}", f"v_add_u32 {v(T[6])}, {s(S_T[3])}, {v(ROWI)}",
                  f"v_min_i32 {v(T[6])}, {s(C_P1)}, {v(T[6])}", f"v_lshlrev_b32 {v(T[6])}, 2, {v(T[6])}",
                  f"global_load_dword {v(SLN[u])}, {v(T[6])}, {s(SLOTS, 2)}"]
        return x

    prefetch = kind not in st.no_prefetch
    if not prefetch and not idle:
        for f in range(NF):
            last[f] = read_frag(f)
    if raw8:
        e(f"v_and_b32 {v(T[6])}, 3, {v(ROWI)}")
        e(f"v_lshlrev_b32 {v(T[6])}, 4, {v(T[6])}")
        e(f"v_xor_b32 {v(T[6])}, {v(KOFF0)}, {v(T[6])}")   # 16 (lane % 16): load block 0 swizzles by the row, lane / 16
    if idle:
        # ---- a wave that has no rows in the tile, or none that sees a key of it: its share of the next tile's loads ----
        if raw8:
            loads = [load_base()] + [load_piece8(u, w) for u in range(upw) for w in range(2)] + [load_exponents()]
        else:
            loads = ([load_base()] if ROWB == 256 else []) + [load_piece(u, w) for u in range(upw) for w in range(2)]
        for piece in loads + ([] if ext else [slot_ids()]):
            for y in piece:
                e(y)
        e("s_waitcnt vmcnt(0)")
        if raw8:
            decode8()
        e("s_barrier")
        end_of_tile()
        return
    # ---- what stands behind the MFMAs, by the number of the MFMA: single instructions, or pieces that stay together ----
    n = 8 * NF
    behind = [[] for _ in range(n)]

    def spread(pieces, first, end):
        """... evenly behind the MFMAs first .. end - 1."""
        for k, piece in enumerate(pieces):
            behind[first + k * (end - first) // len(pieces)] += piece

    def singles(x):
        return [[y] for y in x]
    if raw8:   # (no product while lanes are switched off)
        spread([load_base()] + [load_piece8(u, w) for u in range(upw) for w in range(2)] + [load_exponents()], 0, NF + 2)
        spread([slot_ids()], 2 * NF, n)
    elif not noload:
        loads = (load_base() if ROWB == 256 else []) + [x for u in range(upw) for w in range(2) for x in load_piece(u, w)]
        spread(singles(loads), 0, NF + 2)   # (the probabilities take over their registers)
        if not ext:
            spread(singles(slot_ids()), NF + 2, 2 * NF)
    if masked:
        behind[0].append(f"v_mov_b32 {v(NEGINF)}, 0xff800000")
    # probabilities of block 0: of rows 0..15 once their scores are there (MFMA NF - 1), of rows 16..31 (MFMA 2 NF - 1); those of
    # block 1 likewise
    x = [y for idx in range(8) for y in exp_piece(SC0, PB0, idx)] + [convert()]
    spread(singles(x), NF + 2, 4 * NF - 3)
    behind[4 * NF - 3].append((SC0, PB0))
    if masked:
        behind[4 * NF - 3] += [f"v_subrev_u32 {v(LIM[rb])}, 32, {v(LIM[rb])}" for rb in range(2)]
    x = [y for idx in range(8) for y in exp_piece(SC1, PB1, idx)] + [convert()]
    spread(singles(x), 4 * NF - 2, 6 * NF - 3)
    behind[6 * NF - 3].append((SC1, PB1))
    # ---- the products: per phase, the fragments with rows 0..15, then again with rows 16..31; a buffer is free then and takes the
    # fragment of the next phase that has its number ----
    for i in range(n):
        ph, rb, f = i // (2 * NF), i // NF % 2, i % NF
        g = ph * NF + f
        if i == 4 * NF:
            check_sums(SC0, "Lover1")
        if i == 6 * NF:
            check_sums(SC1, "Lover2")
        if i == 7 * NF and prefetch:
            # this wave's part of the next tile has landed, and so has everyone else's; nobody has a read of this one under way
            assert not st.lds, st.lds
            e("s_waitcnt vmcnt(0)")
            e("s_barrier")
        if rb == 0 and f % 2 == 0:
            st.wait_lds(last[g + 1])
        buf = v(FR[f], 4)
        if ph < 2:
            sl, kb = divmod(f, 2)
            d = v((SC0, SC1)[ph] + 4 * (2 * kb + rb), 4)
            mfma(d, buf, v(Q[rb][sl], 4), d if sl else "0")
        else:
            d = v(ACC[rb][f], 4)
            mfma(d, buf, v((PB0, PB1)[ph - 2] + 4 * rb, 4), d)
        if rb == 1 and ph < 3:
            last[g + NF] = read_frag(g + NF)
        elif rb == 1 and prefetch:
            read_frag(f, there)
        for y in behind[i]:
            if isinstance(y, tuple):
                sum_products(*y)
            else:
                e(y)
    if not prefetch:
        assert not st.lds, st.lds
        e("s_waitcnt vmcnt(0)")
        if raw8:
            decode8()
        if kind not in st.no_barrier:
            e("s_barrier")
    end_of_tile()


KINDS = ["pool", "ext", "pool64", "plain", "masked", "pool8", "pool_idle", "ext_idle", "pool64_idle", "pool8_idle"]   # mode operand = 1 + index
MODE = 50                                                # scalar register of the mode operand


def registers(operand):
    """{"v7", ...} for v7, v[4:7], s[72:73]; vcc; nothing for anything else."""
    m = re.fullmatch(r"-?([vs])(?:(\d+)|\[(\d+):(\d+)\])", operand)
    if not m:
        return {operand} if operand in ("vcc", "m0") else set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {f"{m[1]}{i}" for i in range(lo, hi + 1)}


def check_waits(kind, lines):
    """Tiles of a kind in a row: nothing reads a result before it may (the wait states above).  Time in cycles, four an instruction; an
    MFMA waits for the pipe, which the one before holds for sixteen; what other waves do only adds to it."""
    now, pipe, n = 0, 0, 0
    made = {}   # register -> (instruction that wrote it, its number, when it was issued)
    for text in lines:
        op, _, rest = text.partition(" ")
        args = [registers(a.split()[0]) for a in rest.split(", ") if a]
        if op in ("s_waitcnt", "s_barrier") or op.startswith("s_cbranch"):
            continue
        if op == "s_nop":
            now, n = now + 4 * (int(rest) + 1), n + int(rest) + 1
            continue
        stores = op.startswith(("ds_write", "global_load_lds"))
        reads = set().union(*args) if stores else set().union(*args[1:]) if len(args) > 1 else set()
        if op.startswith("global_load_lds"):
            reads.add("m0")
        if op.startswith("v_mfma"):
            now = max(now, pipe)
            pipe = now + 16
            reads -= args[0]   # (an accumulator that goes on)
        for reg in reads & made.keys():
            by, at, when = made[reg]
            if by.startswith("v_mfma") and op.startswith("v_") and not op.startswith("v_mfma"):
                assert now - when >= 36, (kind, text, now - when)
            wait = 1 if by.startswith("v_exp") or (reg == "m0" and op.startswith("global_load_lds")) else 0
            if "_dpp" in op and reg in args[1] and by.startswith("v_"):   # (the operand that is broadcast)
                wait = 2
            if by.startswith("v_cmp") and op.startswith("v_cndmask"):
                wait = 2
            assert n - at > wait, (kind, text, by, n - at)
        if not stores and args:
            for reg in args[0]:
                made[reg] = (op, n, now)
        now, n = now + 4, n + 1


def gen(upw, kinds, no_barrier=()):
    """All kinds of run in one statement (one set of register constraints for the compiler to meet), chosen by the mode
    operand.  Labels of a kind carry its name; Lover1 / Lover2 / Ldone are common.  A tile of a kind in no_barrier ends
    once this wave's loads have landed, and the caller brings the workgroup together (it has work to do on what landed)."""
    st = Stream()
    st.no_barrier = no_barrier
    # (pool8: the next tile is no bfloat16 yet when the last products of this one begin)
    st.no_prefetch = tuple(no_barrier) + ("pool8",) + tuple(k for k in KINDS if k.endswith("_idle"))
    e = st.emit
    end = "%="
    # ---- entry: LDS read addresses in ring slot 0 (the operands give those of the slot that holds the tile at P0) ----
    e(f"s_lshl_b32 {s(S_T[0])}, {s(RING)}, {STAGEB.bit_length() - 1}")
    e(f"v_subrev_u32 {v(KRD[0])}, {s(S_T[0])}, {v(KRD0)}")
    e(f"v_subrev_u32 {v(VRD[0])}, {s(S_T[0])}, {v(VRD0)}")
    for k in range(1, KS):
        e(f"v_xor_b32 {v(KRD[k])}, {64 * k}, {v(KRD[0])}")
    for b in range(1, NB):
        e(f"v_xor_b32 {v(VRD[b])}, {32 * b}, {v(VRD[0])}")
    # (ones in the first row only: the sum of a query row then comes out in one of the four lanes that share it, zeros in the others)
    e(f"v_mbcnt_lo_u32_b32 {v(T[2])}, -1, 0")
    e(f"v_mbcnt_hi_u32_b32 {v(T[2])}, -1, {v(T[2])}")
    e(f"v_and_b32 {v(T[2])}, 15, {v(T[2])}")
    e(f"v_mov_b32 {v(T[3])}, {ONES}")
    e(f"v_cmp_eq_u32 vcc, 0, {v(T[2])}")
    e("s_nop 1")
    for k in range(4):
        e(f"v_cndmask_b32 {v(ONE + k)}, 0, {v(T[3])}, vcc")
    if ROWB == 256:
        # lane 16 j + u: what the swizzle of load block u differs by from that of block 0, K: 64 u, V: v_swizzle(u); ROWI holds u in
        # its bits 2 and 3
        e(f"v_and_b32 {v(T[2])}, 12, {v(ROWI)}")
        e(f"v_lshlrev_b32 {v(SWZ[0])}, 4, {v(T[2])}")
        e(f"v_and_b32 {v(T[2])}, 4, {v(ROWI)}")
        e(f"v_and_b32 {v(T[3])}, 8, {v(ROWI)}")
        e(f"v_lshlrev_b32 {v(T[2])}, 3, {v(T[2])}")
        e(f"v_lshl_or_b32 {v(SWZ[1])}, {v(T[3])}, 1, {v(T[2])}")
    e(f"s_mov_b32 {s(STATUS)}, 0")
    for kind in kinds[1:]:
        e(f"s_cmp_eq_u32 {s(MODE)}, {KINDS.index(kind) + 1}")
        e(f"s_cbranch_scc1 Lkind_{kind}{end}")
    for kind in kinds:
        uid = f"_{kind}{end}"
        e(f"Lkind{uid}:")
        if kind in ("pool8", "pool8_idle"):
            # lanes that fetch the codes of a row (the first eight of every sixteen); lanes that fetch exponents (the first four)
            e(f"s_mov_b32 {s(MASKS[0])}, 0x00ff00ff")
            e(f"s_mov_b32 {s(MASKS[0] + 1)}, 0x00ff00ff")
            e(f"s_mov_b32 {s(MASKS[1])}, 0x000f000f")
            e(f"s_mov_b32 {s(MASKS[1] + 1)}, 0x000f000f")
        st.kind_end = end
        # the loop body is written out for both ring slots: every LDS offset is an immediate; the first tile's first fragments
        e(f"s_cmp_eq_u32 {s(RING)}, 0")
        e(f"s_cbranch_scc0 Lin1{uid}")
        for ring in range(2):
            e(f"Lin{ring}{uid}:")
            if kind not in st.no_prefetch:
                for f in range(NB):
                    sl, kb = divmod(f, 2)
                    off = ring * STAGEB + kb * 16 * ROWB
                    e(f"ds_read_b128 {v(FR[f], 4)}, {v(KRD[sl])}" + (f" offset:{off}" if off else ""))
            e(f"s_branch Lring{ring}{uid}")
        body = []
        for ring in range(2):
            e(f"Lring{ring}{uid}:")
            st.lds = list(range(st.next_id, st.next_id + (0 if kind in st.no_prefetch else NB)))
            st.next_id += len(st.lds)
            at = len(st.lines)
            tile(st, kind, ring, upw)
            body.append(st.lines[at:])
            e(f"s_cbranch_scc0 Ldone{end}" if ring == 0 else f"s_cbranch_scc1 Lring0{uid}")
        check_waits(kind, body[0] + body[1] + body[0])
        e(f"s_branch Ldone{end}")
    e(f"Lover1{end}:")
    e(f"s_mov_b32 {s(STATUS)}, 1")
    e(f"s_branch Ldone{end}")
    e(f"Lover2{end}:")
    e(f"s_mov_b32 {s(STATUS)}, 2")               # the sum of block 0 is in L already
    e(f"Ldone{end}:")
    e("s_nop 7")                                 # (the last MFMAs, before anything reads the accumulators)
    e("s_waitcnt vmcnt(0) lgkmcnt(0)")           # prefetched fragments and slot ids of a run that was left early
    return st.lines


def emit(name, D, kinds, no_barrier=()):
    shape(D)
    lines = gen(UPW, kinds, no_barrier)
    kv8 = "pool8" in kinds
    body = "\n".join(f'        "{ln}\\n\\t"' for ln in lines)
    free = (set(range(FIRST_V, min(Q[1]))) - set(SLN) - set(L) - set(NEGM) - {KOFF0, VOFF0, ROWI, KRD0, VRD0} - set(LIM))
    clob = ([f"v{i}" for i in sorted(free)] + [f"s{i}" for i in S_T] +
            [f"s{i}" for i in range(MASKS[0], MASKS[1] + 2)] + ["vcc", "scc", "memory"] + (["exec"] if kv8 else []))
    clobbers = ", ".join(f'"{c}"' for c in clob)
    sln = ", ".join(f'"+{{v{SLN[u]}}}"(sl_next[{u}])' for u in range(len(SLN)))
    acc_ops = ",\n          ".join(", ".join(f'"+{{v[{ACC[rb][b]}:{ACC[rb][b] + 3}]}}"(acc[{rb}][{b}])' for b in range(NB)) for rb in range(2))
    q_ops = ", ".join(f'"{{v[{Q[rb][0]}:{Q[rb][0] + 4 * KS - 1}]}}"(q{rb})' for rb in range(2))
    rows = ", ".join(f'"+{{v{L[rb]}}}"(l_run[{rb}]), "+{{v{LIM[rb]}}}"(lim{rb})' for rb in range(2))
    negm = ", ".join(f'"{{v{NEGM[rb]}}}"(neg_m{rb})' for rb in range(2))
    return f'''
// head dimension {D}: a wave loads {UPW} blocks of a tile
__device__ __forceinline__ void {name}(int mode, f32x4 (&acc)[2][{NB}], const bf16x{8 * KS}& q0, const bf16x{8 * KS}& q1,
                                       float (&l_run)[2], float neg_m0, float neg_m1, int32_t (&sl_next)[{len(SLN)}],
                                       unsigned k_rd0, unsigned v_rd0, unsigned ld_koff0, unsigned ld_voff0, int row_in_tile,
                                       int& p0, int& ring, int& status, int p_end, const void* slots, const void* base_k,
                                       const void* base_v, int lim0, int lim1, const i32x8& c, const i32x4& c2{", unsigned exp_stage" if kv8 else ""}) {{
    asm volatile(
{body}
        : {acc_ops},
          {rows},
          {sln}, "+{{s40}}"(p0),
          "+{{s41}}"(ring), "={{s42}}"(status)
        : {q_ops}, {negm}, "{{v{KRD0}}}"(k_rd0), "{{v{VRD0}}}"(v_rd0), "{{v{KOFF0}}}"(ld_koff0),
          "{{v{VOFF0}}}"(ld_voff0), "{{v{ROWI}}}"(row_in_tile), "{{s43}}"(p_end), "{{s[44:45]}}"(slots), "{{s[46:47]}}"(base_k),
          "{{s[48:49]}}"(base_v), "{{s[52:59]}}"(c), "{{s[60:63]}}"(c2), "{{s{MODE}}}"(mode){f', "{{s{EXST}}}"(exp_stage)' if kv8 else ""}
        : {clobbers});
}}
'''


HEADER = '''// GENERATED by gen_fast_run.py - do not edit.  Tiles of extend_bf16_kernel as gfx950 assembly with fixed registers; the
// generator describes the schedule.  One statement per kernel holds every kind of tile, so that the compiler meets one
// set of register constraints; the mode operand chooses:
//   1  a run of tiles, the NEXT tile of each wholly in the prefix (its rows come from the pool through slot ids)
//   2  a run of tiles, the next tile wholly in the extend tokens
//   3  as 1 for pools of 4 GB and more (pool rows addressed in 64 bits; base_k / base_v 256-byte aligned)
//   4  one tile, arithmetic only (the caller has issued the next tile's loads)
//   5  as 4 with keys hidden from rows: lim0 / lim1 = how many keys of the tile, counted from the lane's first, its rows see
//   7, 8, 9  runs as 1, 2, 3 of a wave that has nothing to compute in these tiles: its share of the loads only
// (_kv8, for the fp8 pool: modes 2, 4, 5, 8 and
//   6  a run of tiles, the next tile of each wholly in the prefix: its rows arrive as codes and row exponents and are
//      turned into bfloat16 in LDS once they have landed; base_k / base_v then point at the codes, c[2] is the page
//      stride of the codes in bytes, c[5] the page stride of the row exponents, c[6] the distance from a K row's
//      exponent to its V row's, c2[0..1] the address of the KV head's row exponents, exp_stage the LDS address of the
//      wave's staging area for them;
//   10 the same of a wave that has nothing to compute;
// a single tile (4, 5) ends without the workgroup barrier - the caller decodes the pool rows that have landed first.)
//
// Operands, index or suffix 0 / 1 for the wave's rows 0..15 / 16..31: acc output accumulators, by head-dim block of 16; q the query
// fragments (k-slices of 32); l_run this lane's share of the row sum; neg_m minus the running maximum; sl_next the pool
// slots of this lane's rows of the next tile (updated to those of the tile after the last one done): at head dimension 128 of the
// one whose place it works out (load_base() in the generator), at 64 of those it loads;
// k_rd0 / v_rd0 LDS read addresses (k-slice 0; head-dim block 0, first 16 keys) in the ring slot of the tile at p0;
// ld_koff0 / ld_voff0 byte offsets inside a K / V row of this lane's 16 bytes of load block 0; row_in_tile that row of
// the tile (64: the one it loads in block 0); p0 first key of the tile (advanced by 64 per tile done); ring its ring slot;
// status 0 = ran to p_end, 1 / 2 = the tile at p0 outgrew the running maximum in key block 0 / 1 (see the kernel);
// slots the request's slot ids; base_k / base_v where K / V rows are fetched from; lim0 / lim1 see mode 5 (scratch otherwise);
// c = {page shift, page mask, page stride in bytes (mode 3: in rows of 256 bytes), num_slots - 1, P - 1, extend token
// stride in bytes, kv_hi - 1 - P, LDS address of this wave's load block 0 in ring slot 0}; c2 = {128, 192, P, bits of
// scale * log2(e)}.
'''


def main():
    here = os.path.dirname(os.path.abspath(__file__))
    text = (HEADER + emit("fast_tiles_d128", 128, ["pool", "ext", "pool64", "plain", "masked", "pool_idle", "ext_idle", "pool64_idle"]) +
            emit("fast_tiles_d128_kv8", 128, ["pool8", "ext", "plain", "masked", "pool8_idle", "ext_idle"], no_barrier=("plain", "masked")) +
            emit("fast_tiles_d64", 64, ["pool", "ext", "plain", "masked", "pool_idle", "ext_idle"]))
    path = os.path.join(here, "fast_run.inc")
    old = open(path).read() if os.path.exists(path) else None
    if old != text:
        open(path, "w").write(text)
    return path


if __name__ == "__main__":
    print(main())
