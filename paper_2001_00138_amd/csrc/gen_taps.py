#!/usr/bin/env python3
"""Generates the inner loop of the tap-product kernel (kernel_taps.hip) as one inline-assembly
statement for gfx950.

What the loop computes: for one wavefront, the filters of its group(s) and one chunk of staged
input channels, the convolution of a 16 x 16 tile of input pixels.  A kept kernel is ONE
``v_mfma_f32_4x4x1_16b_f32`` per 64 pixels: the outer product of its four weights (matrix A,
broadcast to all sixteen blocks of the instruction) and the pixels of its input channel (matrix
B, one per lane) is added to four accumulator registers, one per tap - D[tap] += weight[tap] *
pixel, not yet shifted to the output pixel it belongs to.  All kernels of one filter that
share a pattern accumulate into the same registers; only when the pattern changes are the four
tap sums shifted and added to the filter's output rows ("flush").  The shift is the tap's
position: a lane holds four consecutive rows of one column, so a vertical shift is a choice of
register (rows that leave the lane's four go to two carry registers) and a horizontal one is left
for later: there are three sets of rows, one per column of the 3 x 3 window, which are shifted
against each other (DPP row shifts) and added up when the filter ends, when the carries are
handed to the lanes above as well.  A flush is then sixteen adds on vector registers alone,
which issue at twice the rate of adds with a DPP operand.

Stream (layout.hpp, ``Taps``): batches of 16 kernels; a record per kernel (channel in the chunk,
pattern, end-of-segment and end-of-filter marks) read over the scalar data path one batch ahead,
and 64 weights per batch, one per lane, in one vector register: the instruction's ABID field,
fixed for each of the sixteen unrolled bodies, picks the kernel's four.

Registers are fixed at generation time above ``vbase`` (the compiler keeps the output
accumulators below it).  Nothing is written through the scalar data path.
"""

import os
import sys

from gen_dispatch import universe

GROUP = 8                      # filters of one stream
TILE = 16                      # rows and columns of a tile
FLUSH_BYTES = 256              # bytes per flush block (one per pattern, and an empty one)
END_BYTES = 512                # bytes per end-of-filter block

# scalar registers
REC = (36, 52)                 # two sets of 16 records
BASE, TGT, RET, RET2, ENDP, SP, WP, TMP = 68, 70, 72, 74, 76, 78, 80, 82
S_CLOBBER = (36, 82)
# vector registers, relative to vbase; behind the pixels' quads come A, P and ADDR
D, X = 0, 16


def buffers(ahead):
    """Quads for pixels, those on their way and one that the matrix cores still read: a power of two, since the
    bodies of a batch of 16 kernels have theirs fixed."""
    return 1 << ahead.bit_length()


def registers(ahead):
    """First of A, P and ADDR, and the number of all."""
    a = X + 4 * buffers(ahead)
    return a, a + 2, a + 20, a + 21


def program(F, vbase, ahead):
    """Assembly lines.  Operands: %[o<f>_<r>] output rows of filter f (r = 0..3), %[lane] LDS byte
    address of the lane's 16 bytes in channel 0 (16 * lane: the chunk starts at LDS address 0),
    %[rec] / %[wp] addresses of the first kernel's record / weights, %[first] first of the
    GROUP filters whose stream this is (0 where a wavefront has fewer).  ``ahead``: kernels whose pixels are on
    their way from LDS."""
    lines = []
    asm = lines.append
    group, nbuf = min(F, GROUP), buffers(ahead)
    A, P, ADDR, _ = registers(ahead)

    def v(i):
        return f"v{vbase + i}"

    def v4(i):
        return f"v[{vbase + i}:{vbase + i + 3}]"

    def align(log2):
        asm(f".p2align {log2}")

    def fit(label, size):
        asm(f".if . - {label} > {size}")
        asm('.error "code block larger than its slot"')
        asm(".endif")

    # ---- set-up
    asm(f"s_getpc_b64 s[{BASE}:{BASE + 1}]")
    asm(".Lpc%=:")
    asm(f"s_mul_i32 s{TMP}, %[first], {END_BYTES}")
    asm(f"s_add_u32 s{TMP}, s{TMP}, .Lend0_%=-.Lpc%=")
    asm(f"s_add_u32 s{ENDP}, s{BASE}, s{TMP}")
    asm(f"s_addc_u32 s{ENDP + 1}, s{BASE + 1}, 0")
    asm(f"s_add_u32 s{BASE}, s{BASE}, .Lflush0_%=-.Lpc%=")
    asm(f"s_addc_u32 s{BASE + 1}, s{BASE + 1}, 0")
    asm(f"s_mov_b64 s[{SP}:{SP + 1}], %[rec]")
    asm(f"s_mov_b64 s[{WP}:{WP + 1}], %[wp]")

    def fetch(st):
        asm(f"s_load_dwordx16 s[{REC[st]}:{REC[st] + 15}], s[{SP}:{SP + 1}], 0x0")
        asm(f"v_lshrrev_b32 {v(ADDR)}, 2, %[lane]")
        asm(f"global_load_dword {v(A + st)}, {v(ADDR)}, s[{WP}:{WP + 1}]")
        asm(f"s_add_u32 s{SP}, s{SP}, 64")
        asm(f"s_addc_u32 s{SP + 1}, s{SP + 1}, 0")
        asm(f"s_add_u32 s{WP}, s{WP}, 256")
        asm(f"s_addc_u32 s{WP + 1}, s{WP + 1}, 0")

    def read_pixels(rec, buf):
        # the record's low byte is the channel; its marks are shifted out of the address
        asm(f"v_lshl_add_u32 {v(ADDR)}, s{rec}, 10, %[lane]")
        asm(f"ds_read_b128 {v4(X + 4 * buf)}, {v(ADDR)}")

    fetch(0)
    for i in range(18):
        asm(f"v_mov_b32 {v(P + i)}, 0")
    asm("s_waitcnt lgkmcnt(0)")
    for k in range(ahead):
        read_pixels(REC[0] + k, k)
    asm("s_branch .Lk0_0_first_%=")

    # ---- one body per (record set, kernel of the batch, first of a segment or not)
    def body(st, k, first):
        asm(f".Lk{st}_{k}_{'first' if first else 'next'}_%=:")
        if k == 0:
            asm("s_waitcnt vmcnt(0)")                # this batch's weights
            fetch(1 - st)                            # the next batch
        nxt = k + ahead
        if nxt == 16:
            asm("s_waitcnt lgkmcnt(0)")              # the next batch's records
        read_pixels(REC[st] + nxt if nxt < 16 else REC[1 - st] + nxt - 16, nxt % nbuf)
        # LDS reads complete in order; a scalar load still in flight only makes this wait stricter
        asm(f"s_waitcnt lgkmcnt({ahead})")
        for r in range(4):
            c = "0" if first else v4(D + 4 * r)
            asm(f"v_mfma_f32_4x4x1_16b_f32 {v4(D + 4 * r)}, {v(A + st)}, {v(X + 4 * (k % nbuf) + r)}, {c} cbsz:4 abid:{k}")
        asm(f"s_cmp_lt_i32 s{REC[st] + k}, 0")       # end of segment: bit 31
        asm(f"s_cbranch_scc1 .Lseg{st}_{k}_%=")

    for first in (True, False):
        for st in range(2):
            for k in range(16):
                body(st, k, first)
                # falls through to the next kernel of the same segment; a body that ran as the first
                # of its segment goes on in the other copy
                ns, nk = (st, k + 1) if k < 15 else (1 - st, 0)
                if first or (st, k) == (1, 15):
                    asm(f"s_branch .Lk{ns}_{nk}_next_%=")

    # ---- end of a segment: flush by pattern, then the filter's end if it is one
    for st in range(2):
        for k in range(16):
            ns, nk = (st, k + 1) if k < 15 else (1 - st, 0)
            asm(f".Lseg{st}_{k}_%=:")
            asm(f"s_bfe_u32 s{TMP}, s{REC[st] + k}, {14 << 16 | 14}")       # pattern (bits 22..27) * FLUSH_BYTES: bits 14..21 are zero
            asm(f"s_add_u32 s{TGT}, s{BASE}, s{TMP}")
            asm(f"s_addc_u32 s{TGT + 1}, s{BASE + 1}, 0")
            asm(f"s_swappc_b64 s[{RET}:{RET + 1}], s[{TGT}:{TGT + 1}]")
            asm(f"s_bitcmp1_b32 s{REC[st] + k}, 30")             # end of filter
            asm(f"s_cbranch_scc0 .Lk{ns}_{nk}_first_%=")
            asm(f"s_swappc_b64 s[{RET2}:{RET2 + 1}], s[{ENDP}:{ENDP + 1}]")
            asm(f"s_branch .Lk{ns}_{nk}_first_%=")

    # ---- flush blocks, FLUSH_BYTES apart: tap sum of row r -> output row r - kh, column - kw
    for p, taps in enumerate(universe()):
        align(8)
        asm(f".Lflush{p}_%=:")
        asm("s_nop 1")                               # with the scalar instructions before: MFMA result to VALU
        for r in range(4):
            for t, pos in enumerate(taps):
                kh, kw = divmod(pos, 3)
                dst = v(P + 6 * kw + 2 + r - kh)
                asm(f"v_add_f32 {dst}, {v(D + 4 * r + t)}, {dst}")
        asm(f"s_setpc_b64 s[{RET}:{RET + 1}]")
        fit(f".Lflush{p}_%=", FLUSH_BYTES)
    align(8)                                         # kTapNothing: a filter without kernels in this chunk
    asm(f"s_setpc_b64 s[{RET}:{RET + 1}]")

    # ---- end-of-filter blocks, END_BYTES apart
    for f in range(F):
        align(9)
        asm(f".Lend{f}_%=:")
        # rows -2 .. 3 of the lane: the three column sets, shifted against each other
        for kw in (1, 2):
            for i in range(6):
                asm(f"v_add_f32_dpp {v(P + i)}, {v(P + 6 * kw + i)}, {v(P + i)} row_shl:{kw} row_mask:0xf bank_mask:0xf bound_ctrl:0")
        # rows -2 and -1 belong to the lanes sixteen before (the tap sums are free here)
        asm(f"v_lshrrev_b32 {v(ADDR)}, 2, %[lane]")
        asm(f"v_add_u32 {v(ADDR)}, 64, {v(ADDR)}")
        asm(f"v_and_b32 {v(ADDR)}, 0xfc, {v(ADDR)}")
        for i in range(2):
            asm(f"ds_bpermute_b32 {v(D + i)}, {v(ADDR)}, {v(P + i)}")
        for r in range(4):
            asm(f"v_add_f32 %[o{f}_{r}], {v(P + 2 + r)}, %[o{f}_{r}]")
        last = f % group == group - 1
        if not last:
            for i in range(18):
                asm(f"v_mov_b32 {v(P + i)}, 0")
        asm("s_waitcnt lgkmcnt(0)")
        asm("s_mov_b32 exec_hi, 0xffff")             # the last sixteen lanes have nothing below them
        for i in range(2):
            asm(f"v_add_f32 %[o{f}_{2 + i}], {v(D + i)}, %[o{f}_{2 + i}]")
        asm("s_mov_b32 exec_hi, -1")
        if last:
            asm("s_branch .Lexit_%=")
        else:
            asm(f"s_add_u32 s{ENDP}, s{ENDP}, {END_BYTES}")
            asm(f"s_addc_u32 s{ENDP + 1}, s{ENDP + 1}, 0")
            asm(f"s_setpc_b64 s[{RET2}:{RET2 + 1}]")
        fit(f".Lend{f}_%=", END_BYTES)
    asm(".Lexit_%=:")
    asm("s_waitcnt vmcnt(0) lgkmcnt(0)")             # what was fetched ahead
    return lines


def generate(F, vbase, ahead):
    L = []
    emit = L.append
    emit(f"template <> struct TapLoop<{F}> {{")
    emit(f"    static __device__ __forceinline__ void run(float (&o)[{F}][4], unsigned lane_lds,")
    emit("                                               const uint32_t* rec, const float* wp, int first)")
    emit("    {")
    emit("        asm volatile(")
    lines = program(F, vbase, ahead)
    for i in range(0, len(lines), 32):
        text = "\\n".join(s.replace('"', '\\"') for s in lines[i:i + 32])
        emit(f'            "{text}\\n"')
    outs = ", ".join(f'[o{f}_{r}] "+v"(o[{f}][{r}])' for f in range(F) for r in range(4))
    clob = ", ".join([f'"s{i}"' for i in range(S_CLOBBER[0], S_CLOBBER[1] + 1)] +
                     [f'"v{vbase + i}"' for i in range(registers(ahead)[3])])
    emit(f"            : {outs}")
    emit('            : [lane] "v"(lane_lds), [rec] "s"(rec), [wp] "s"(wp), [first] "s"(first)')
    emit(f'            : {clob}, "scc", "memory");')
    emit("    }")
    emit("};")
    return "\n".join(L) + "\n"


# (filters per wavefront, first fixed vector register, kernels ahead).  Three kernels ahead cover the reads where
# four or five wavefronts share a SIMD, and leave 16 filters 128 registers; the wavefronts of few filters are for launches
# that have one or two for each SIMD.
VARIANTS = ((2, 18, 6), (4, 26, 6), (8, 42, 3), (16, 74, 3))


def main(argv):
    out_dir = argv[1]
    os.makedirs(out_dir, exist_ok=True)
    text = "// Generated by gen_taps.py - do not edit.\n" + "".join(generate(*v) for v in VARIANTS)
    path = os.path.join(out_dir, "taps_all.inc")
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as f:
            f.write(text)


if __name__ == "__main__":
    main(sys.argv)
