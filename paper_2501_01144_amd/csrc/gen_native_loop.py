#!/usr/bin/env python3
"""Generator of gemm_native_asm.inc: main loop of gemm_native_kernel (block-scaled
v_mfma_scale_f32_16x16x128_f8f6f4 on FP4 or FP6 operands, see gemm_native.hip).

A workgroup computes 256 x 256 outputs with four waves as 2 x 2, each wave 128 x 128 (8 x 8 tiles of
16 x 16, accumulator tile (i, j) in a[4 (8 i + j) : +3]).  A second form (suffix _H) halves the rows: 128 x 256 per
workgroup, 64 x 128 per wave, for products with few tiles.  W is the instruction's first operand and A its second, so that a
lane holds four neighbouring columns of one row of the result.

One iteration = four blocks (K = 128) = two steps of the packed operands = 64 (32) instructions per wave.  The packed form
(gemm_native.hip, fp6_pack.h) keeps (32 rows, step of two blocks) together; lane (q, c) of a 16 x 16 x 128 instruction
wants block q of row c, which is step q / 2, block q % 2 there, so a lane's LDS address has the stage in it and nothing is laid
out anew.  Both operands arrive

  global -> LDS  direct loads (global_load_lds_dwordx4, whole KiB), two (three) iterations ahead, three (four) slots
                 of two stages in rotation;
                 wave w fetches A tiles 2w, 2w+1, B tiles 2w, 2w+1 (of 32 rows) and scale chunk w; in the 128-row form
                 A tile w, and of an FP6 pair's last KiB both waves of the pair write the same copy;
  LDS -> regs    the wave's operands and scale dwords of iteration d + 1 are read during iteration d (two register sets
                 used alternately);
  one barrier per iteration, two multiplications in: after it every wave's loads of iteration d + 1 have landed and
                 nobody reads the slot that this iteration's loads overwrite.

Where there is nothing new to load any more, the loads read the last step again.  Where the number of steps is
odd the second half of the last iteration is what lies behind (the next tile, or the slack), and A's registers of it and the scales (the
upper 32 lanes) are cleared: FP4 and FP6 have no infinities, so it multiplies to zero.

Why this instruction: the kernel is bound by power, and it takes a tenth less of it than 32 x 32 x 64 for the same products.
Loops of either on registers with operands as they come sustain 6.3 (FP6) and 6.9 PFLOP/s (FP4) with 32 x 32 x 64 at 1.56 and
1.71 GHz, 7.0 and 7.7 with 16 x 16 x 128 at 1.76 and 1.94; neighbouring instructions share an operand (rows of tiles forth and
back), half a per cent.  What it asks for: an instruction takes 16 clocks, and a wave, which is alone on its SIMD, gets one
other short instruction into its shadow.  With two or three behind some and none behind others, addresses rotated between
iterations and a branch taken in each, a step of K = 64 took 885 clocks (FP6); with everything unrolled and spread evenly it
takes 600 (512 without any other work), at 1.48 GHz, against 660 at 1.43 with the larger instruction.  4096 x 4096, K = 8192,
loop alone: FP6 58 -> 52 us, FP4 51.6 -> 46.6.  On operands that are all zero the same loop runs at the full clock, 2.4 GHz.

LDS stage: the chunks of A tiles 0..7 and B tiles 0..7 as in memory (1 KiB per tile for FP4, 3 KiB per pair for FP6) +
4 x 256 bytes of scales (A groups 0, 1, B groups 0, 1).  Per step FP6 moves 25 KB into LDS and 50 KB out of it, 600 clocks at
128 byte/clock: as long as a step takes, so that a clock spared elsewhere in the loop gains nothing.  Registers 4, 5 are kept at
8 bytes per lane: at the 16-byte stride that 12-byte direct loads leave, their reads cost as much as 16-byte ones.  The reads of
scales conflict, two clocks each, four an iteration and wave: the blocks of lanes q and q + 2 lie a stage apart, a multiple
of 256 bytes (that and 16 clocks a group of fp32 results are all conflicts that the counters see).

With operands that the last cache does not hold a step takes as long as its bytes at 60 byte/ns and compute unit, however
early they are asked for (FP6: 128-row form 1.28 times as long, 256 rows 1.07; FP4 1.13 and 1.01): what a compute unit can
have in flight.

Registers (fixed): a[0:255] accumulators; v[40:135] / v[136:231] operand sets (A tile i at +6 i, B tile j at +48 + 6 j);
v[232:239] scale dwords, of either set A's even and odd tiles, B's; v240 / v241 global offsets (operands, scales); v242.. LDS
read addresses; s[60:69] global bases of the wave's five chunks, s70 iteration, s71 iteration before which something is to be
done, s72 / s73 bytes to the next step's operands and scales, s74 / s75 scratch, s76 shift of A's scales (128-row form),
s77..s84 the wave's LDS addresses inside slot 0 (reads: A, B, scales A, B; loads: A, B, scales, the FP6 pair of A in the
128-row form).
"""
import os

FR = [40, 136]
SC = [232, 236]                  # scale dwords of a set: A even, A odd tiles, B even, B odd
VOFF, VSOFF = 240, 241
VBASE = 242                      # LDS read addresses, slots 0 and 1, then the others: operands A, B, scales A, B, registers 4, 5 of A, B
S_BASE, S_VC, S_EVENT, S_GS, S_SS = 60, 70, 71, 72, 73
S_T0, S_T1, S_SHIFT = 74, 75, 76
S_RA, S_RB, S_RSA, S_RSB, S_DA, S_DB, S_DS, S_DA2 = 77, 78, 79, 80, 81, 82, 83, 84


def vr(n, cnt=1):
    return f"v{n}" if cnt == 1 else f"v[{n}:{n + cnt - 1}]"


def sr(n, cnt=1):
    return f"s{n}" if cnt == 1 else f"s[{n}:{n + cnt - 1}]"


class Fmt:
    def __init__(self, fp6, ta=4):
        self.fp6 = fp6
        self.ta = ta                                 # A tiles of 32 rows per wave: 4 (256-row workgroup) or 2 (128)
        self.ni = 2 * ta                             # A tiles of 16 rows
        self.regs = 6 if fp6 else 4
        self.tile = 1536 if fp6 else 1024            # LDS bytes per 32-row tile and stage
        self.stage = (2 * ta + 8) * self.tile + 1024
        self.gstride = 3072 if fp6 else 1024         # global bytes per (pair of tiles, step) / (tile, step)
        self.code = 2 if fp6 else 4                  # cbsz / blgp
        # direct loads per wave and step: A, B, scales
        self.per_step = (3 if ta == 4 else 2) + 3 + 1 if fp6 else ta // 2 + 2 + 1
        self.behind = []                             # code out of the loop's way
        self.slots = 3 if fp6 and ta == 4 else 4     # of two stages (FP6: 6 x 25 KiB or 8 x 19 KiB, FP4: 8 x 17 or 13 KiB)


def frag_reads(f, p, slot):
    """LDS reads of the operands in `slot` into register set p, in the order in which they are wanted."""
    va, vb, vsa, vsb, va2, vb2 = (VBASE + 6 * (slot >> 1) + i for i in range(6))
    o, at = [], (slot & 1) * 2 * f.stage
    scales = [f"ds_read_b32 {vr(SC[p] + i)}, {vr(v)} offset:{at + 64 * (i & 1)}" for i, v in ((0, vsa), (1, vsa), (2, vsb), (3, vsb))]
    for side, v, v2 in ((1, vb, vb2), (0, va, va2)):
        for t in range(8 if side else f.ni):
            r = FR[p] + 48 * side + 6 * t
            t32, half = t >> 1, t & 1
            if f.fp6:
                pair = (t32 >> 1) * 3072
                o.append(f"ds_read_b128 {vr(r, 4)}, {vr(v)} offset:{at + pair + (t32 & 1) * 1024 + half * 256}")
                o.append(f"ds_read_b64 {vr(r + 4, 2)}, {vr(v2)} offset:{at + pair + 2048 + (t32 & 1) * 512 + half * 256}")
            else:
                o.append(f"ds_read_b128 {vr(r, 4)}, {vr(v)} offset:{at + t32 * f.tile + half * 256}")
        if side:
            o += scales
    return o


def shift_scales(f, p):
    """128-row form: both row halves of the workgroup share one scale dword, bytes 2 wm, 2 wm + 1"""
    return [f"v_lshrrev_b32 {vr(SC[p] + i)}, {sr(S_SHIFT)}, {vr(SC[p] + i)}" for i in (0, 1)] if f.ta == 2 else []


def dma_groups(f, stage):
    """Direct loads of one step of this wave into `stage`, as groups (m0 setup, [loads that use it]).  An instruction offset
    applies to the global and to the LDS address alike, so the loads of one FP6 chunk share one m0."""
    o = []

    def group(dst, base, offsets, disp=0):
        at = f"{vr(VOFF)}, {sr(S_BASE + 2 * base, 2)}"
        o.append((f"s_add_u32 m0, {sr(dst)}, {stage * f.stage + disp}",
                  [f"global_load_lds_dwordx4 {at}" + (f" offset:{x}" if x else "") for x in offsets]))

    if f.fp6:
        if f.ta == 4:
            group(S_DA, 0, (0, 1024, 2048))
        else:
            group(S_DA, 0, (0,))
            group(S_DA2, 1, (2048,))
        group(S_DB, 2, (0, 1024, 2048))
    else:
        for k in range(f.ta // 2):
            group(S_DA, k, (0,), k * f.tile)
        for k in range(2):
            group(S_DB, 2 + k, (0,), k * f.tile)
    o.append((f"s_add_u32 m0, {sr(S_DS)}, {stage * f.stage}", [f"global_load_lds_dword {vr(VSOFF)}, {sr(S_BASE + 8, 2)}"]))
    return o


def next_step():
    return [f"v_add_u32 {vr(VOFF)}, {sr(S_GS)}, {vr(VOFF)}", f"v_add_u32 {vr(VSOFF)}, {sr(S_SS)}, {vr(VSOFF)}"]


def mfma(f, p, i, j):
    k = 8 * i + j
    acc = f"a[{4 * k}:{4 * k + 3}]"
    a = vr(FR[p] + 6 * i, f.regs)
    b = vr(FR[p] + 48 + 6 * j, f.regs)
    bi, bj = i >> 1, j >> 1               # bytes of the scale dwords
    return (f"v_mfma_scale_f32_16x16x128_f8f6f4 {acc}, {b}, {a}, {acc}, {vr(SC[p] + 2 + (j & 1))}, {vr(SC[p] + (i & 1))} "
            f"op_sel:[{bj & 1},{bi & 1},0] op_sel_hi:[{bj >> 1},{bi >> 1},0] cbsz:{f.code} blgp:{f.code}")


BARRIER_AT = 2                   # multiplications before the barrier


def iteration(f, u):
    """Iteration u (mod the unrolled ones): multiplies register set u % 2, reads the operands of the next iteration from its slot,
    loads this one's slot, which has been read.  One other instruction behind each multiplication: the next is issued 16 clocks
    later, and two or more take longer than that."""
    p, slot = u % 2, u % f.slots
    order = [(i, j if i % 2 == 0 else 7 - j) for i in range(f.ni) for j in range(8)]
    n = len(order)
    reads = frag_reads(f, 1 - p, (slot + 1) % f.slots)
    items = [((r + 0.5) / len(reads), "", text) for r, text in enumerate(reads)]
    dma = []
    for half in (0, 1):
        for m0, loads in dma_groups(f, 2 * slot + half):
            for ld in loads:
                dma.append((m0, ld))
                m0 = ""
        dma += [("", text) for text in next_step()]
    items += [(d / len(dma), m0, text) for d, (m0, text) in enumerate(dma)]
    items.sort(key=lambda x: x[0])
    before, behind = [[] for _ in order], [[] for _ in order]           # of the multiplications
    for x, (_, m0, text) in enumerate(items):
        k = BARRIER_AT + x * (n - BARRIER_AT) // len(items)
        if m0:
            (before[k] if not behind[k] else behind[k]).append(m0)
            if behind[k]:
                behind[k].append("s_nop 0")                             # (m0 needs one instruction before its use)
        behind[k].append(text)
    behind[1].append(f"s_add_u32 {sr(S_VC)}, {sr(S_VC)}, 1")
    # B, the scales and A's first tile are there; A's others may be on their way until the barrier
    o = []
    for k, (i, j) in enumerate(order):
        if k == BARRIER_AT:
            # the loads of the next iteration have landed; those of the iterations after it may be pending
            o += [f"s_waitcnt vmcnt({(f.slots - 2) * 2 * f.per_step}) lgkmcnt(0)", "s_barrier"]
        o += before[k] + [mfma(f, p, i, j)] + behind[k]
    return o + next_operands(f, 1 - p, 20 + u)


def next_operands(f, p, label):
    """The operands of register set p, as far as the first row of tiles needs them, and what is to be done in few iterations, out of the loop's
    way (a branch that is taken costs 40 clocks): leave it, stop the loads, clear what is not there."""
    f.behind += [f"{label}:", f"s_cmp_eq_u32 {sr(S_VC)}, %[iters]", "s_cbranch_scc1 99f",
                 # from here on the last step that was loaded is loaded again
                 f"s_cmp_eq_u32 {sr(S_GS)}, 0", f"s_cbranch_scc1 {label + 20}f",
                 f"v_subrev_u32 {vr(VOFF)}, {sr(S_GS)}, {vr(VOFF)}", f"v_subrev_u32 {vr(VSOFF)}, {sr(S_SS)}, {vr(VSOFF)}",
                 f"s_mov_b32 {sr(S_GS)}, 0", f"s_mov_b32 {sr(S_SS)}, 0",
                 f"{label + 20}:", f"s_min_u32 {sr(S_EVENT)}, %[half], %[iters]",
                 f"s_cmp_eq_u32 {sr(S_VC)}, %[half]", f"s_cbranch_scc0 {label + 40}b",
                 # the last iteration of an odd number of steps: there is no second step
                 f"s_mov_b32 {sr(S_EVENT)}, %[iters]", "s_waitcnt lgkmcnt(0)", "s_mov_b32 exec_lo, 0"]
    f.behind += [f"v_mov_b32 {vr(FR[p] + 6 * t + r)}, 0" for t in range(f.ni) for r in range(f.regs)]
    f.behind += [f"v_mov_b32 {vr(SC[p] + i)}, 0x7f7f7f7f" for i in range(4)]
    f.behind += ["s_mov_b32 exec_lo, -1", f"s_branch {label + 40}b"]
    return [f"s_waitcnt lgkmcnt({(f.ni - 1) * (2 if f.fp6 else 1)})"] + shift_scales(f, p) + \
           [f"s_cmp_eq_u32 {sr(S_VC)}, {sr(S_EVENT)}", f"s_cbranch_scc1 {label}f", f"{label + 40}:"]


def entry(f):
    o = [f"v_accvgpr_write_b32 a{n}, 0" for n in range(64 * f.ta)]
    # global bases: FP4 A tiles 2w, 2w+1 and B tiles 2w, 2w+1 (each tile holds `tstride` bytes); FP6 A pair w and B
    # pair w, or in the 128-row form A tile w and (second base) its pair; scale chunk
    o += [f"s_mov_b32 {sr(S_BASE)}, %[alo]", f"s_mov_b32 {sr(S_BASE + 1)}, %[ahi]",
          f"s_add_u32 {sr(S_BASE + 2)}, %[alo], %[tstride]", f"s_addc_u32 {sr(S_BASE + 3)}, %[ahi], 0",
          f"s_mov_b32 {sr(S_BASE + 4)}, %[blo]", f"s_mov_b32 {sr(S_BASE + 5)}, %[bhi]",
          f"s_add_u32 {sr(S_BASE + 6)}, %[blo], %[tstride]", f"s_addc_u32 {sr(S_BASE + 7)}, %[bhi], 0",
          f"s_mov_b32 {sr(S_BASE + 8)}, %[slo]", f"s_mov_b32 {sr(S_BASE + 9)}, %[shi]"]
    # the wave's LDS addresses inside slot 0: wm = wv >> 1, wn = wv & 1
    offb, offs = 2 * f.ta * f.tile, (2 * f.ta + 8) * f.tile
    o += [f"s_lshr_b32 {sr(S_T0)}, %[wv], 1", f"s_and_b32 {sr(S_T1)}, %[wv], 1",
          f"s_mul_i32 {sr(S_RA)}, {sr(S_T0)}, {f.ta * f.tile}", f"s_add_u32 {sr(S_RA)}, {sr(S_RA)}, %[lds]",
          f"s_mul_i32 {sr(S_RB)}, {sr(S_T1)}, {4 * f.tile}", f"s_add_u32 {sr(S_RB)}, {sr(S_RB)}, {offb}",
          f"s_add_u32 {sr(S_RB)}, {sr(S_RB)}, %[lds]"]
    if f.ta == 4:
        o += [f"s_lshl_b32 {sr(S_RSA)}, {sr(S_T0)}, 8", f"s_add_u32 {sr(S_RSA)}, {sr(S_RSA)}, {offs}"]
    else:
        o += [f"s_mov_b32 {sr(S_RSA)}, {offs}"]
    o += [f"s_add_u32 {sr(S_RSA)}, {sr(S_RSA)}, %[lds]",
          f"s_lshl_b32 {sr(S_RSB)}, {sr(S_T1)}, 8", f"s_add_u32 {sr(S_RSB)}, {sr(S_RSB)}, {offs + 512}",
          f"s_add_u32 {sr(S_RSB)}, {sr(S_RSB)}, %[lds]",
          f"s_mul_i32 {sr(S_DA)}, %[wv], {(f.ta // 2) * f.tile}", f"s_add_u32 {sr(S_DA)}, {sr(S_DA)}, %[lds]",
          f"s_mul_i32 {sr(S_DB)}, %[wv], {2 * f.tile}", f"s_add_u32 {sr(S_DB)}, {sr(S_DB)}, {offb}",
          f"s_add_u32 {sr(S_DB)}, {sr(S_DB)}, %[lds]"]
    if f.fp6 and f.ta == 2:           # A tile w inside pair w / 2: 1 KiB apart, in memory and in LDS
        o += [f"s_lshl_b32 {sr(S_DS)}, {sr(S_T1)}, 10",
              f"s_sub_u32 {sr(S_BASE + 2)}, %[alo], {sr(S_DS)}", f"s_subb_u32 {sr(S_BASE + 3)}, %[ahi], 0",
              f"s_mul_i32 {sr(S_DA2)}, {sr(S_T0)}, 3072", f"s_add_u32 {sr(S_DA2)}, {sr(S_DA2)}, %[lds]",
              f"s_add_u32 {sr(S_DA)}, {sr(S_DA2)}, {sr(S_DS)}"]
    if f.ta == 4:
        o += [f"s_lshl_b32 {sr(S_DS)}, %[wv], 8"]
    else:                             # scale chunks: wave 0 and 1 -> the A group (slot 0), waves 2, 3 -> B groups (slots 2, 3)
        o += [f"s_cmp_lt_u32 %[wv], 2", f"s_cselect_b32 {sr(S_DS)}, 0, %[wv]", f"s_lshl_b32 {sr(S_DS)}, {sr(S_DS)}, 8"]
    o += [f"s_add_u32 {sr(S_DS)}, {sr(S_DS)}, {offs}", f"s_add_u32 {sr(S_DS)}, {sr(S_DS)}, %[lds]"]
    # lane (q, c): block q % 2 of row c in stage q / 2 of the slot
    bases = [(S_RA, "%[r16]"), (S_RB, "%[r16]"), (S_RSA, "%[r4]"), (S_RSB, "%[r4]")]
    if f.fp6:
        bases += [(S_RA, "%[r8]"), (S_RB, "%[r8]")]
    for i, (s, lane) in enumerate(bases):
        o += [f"v_add_u32 {vr(VBASE + i)}, {sr(s)}, {lane}", f"v_add_u32 {vr(VBASE + 6 + i)}, {4 * f.stage}, {vr(VBASE + i)}"]
    o += [f"s_mov_b32 {sr(S_VC)}, 0", f"s_mov_b32 {sr(S_GS)}, {f.gstride}", f"s_movk_i32 {sr(S_SS)}, 0x100",
          f"s_lshl_b32 {sr(S_SHIFT)}, %[wv], 3", f"s_and_b32 {sr(S_SHIFT)}, {sr(S_SHIFT)}, 16",          # 16 wm
          # the first iteration that loads nothing new
          f"s_max_u32 {sr(S_EVENT)}, %[iters], {f.slots}", f"s_sub_u32 {sr(S_EVENT)}, {sr(S_EVENT)}, {f.slots}",
          f"v_mov_b32 {vr(VOFF)}, %[g16]", f"v_mov_b32 {vr(VSOFF)}, %[g4]"]
    # pipeline fill: all slots, or as many as there are iterations (K = 32, 2048 x 2048: FP6 8.3 -> 7.5 us of fp32 and 6.3 -> 5.6 of bf16, FP4
    # 7.7 -> 7.3 and 5.7 -> 5.3; from as many iterations as slots on the same)
    for stage in range(2 * f.slots):
        if stage % 2 == 0 and stage:
            o += [f"s_cmp_eq_u32 %[iters], {stage // 2}", "s_cbranch_scc1 70f"]
        for m0, loads in dma_groups(f, stage):
            o += [m0, "s_nop 0"] + loads
        o += next_step()
    # the first iteration's operands into set 0
    o += [f"s_waitcnt vmcnt({(f.slots - 1) * 2 * f.per_step})", "71:", "s_barrier"]
    f.behind += ["70:", "s_waitcnt vmcnt(0)", "s_branch 71b"]
    return o + frag_reads(f, 0, 0) + next_operands(f, 0, 19)


def main_loop(f):
    o = entry(f)
    o.append("80:")
    for u in range(6 if f.slots == 3 else 4):        # both register sets and all slots
        o += iteration(f, u)
    o += ["s_branch 80b"] + f.behind
    o += ["99:", "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_nop 15", "s_nop 15", "s_nop 15", "s_nop 15"]
    return o


def c_string(lines):
    return " \\\n".join(f'    "{l}\\n\\t"' for l in lines)


def main():
    here = os.path.dirname(os.path.abspath(__file__))
    parts = ["// Generated by gen_native_loop.py -- do not edit; see that file for the register map.\n"]
    parts.append("#define DFP4_NATIVE_LOOP_FP4 \\\n" + c_string(main_loop(Fmt(False))) + "\n")
    parts.append("#define DFP4_NATIVE_LOOP_FP6 \\\n" + c_string(main_loop(Fmt(True))) + "\n")
    parts.append("#define DFP4_NATIVE_LOOP_FP4_H \\\n" + c_string(main_loop(Fmt(False, 2))) + "\n")
    parts.append("#define DFP4_NATIVE_LOOP_FP6_H \\\n" + c_string(main_loop(Fmt(True, 2))) + "\n")
    for g in range(16):
        rd = [f"v_accvgpr_read_b32 %{i}, a{16 * g + i}" for i in range(16)]
        parts.append(f"#define DFP4_NATIVE_ACC_READ_{g} \\\n" + c_string(rd) + "\n")
    vclob = ", ".join(f'"v{n}"' for n in range(40, 254))
    aclob = ", ".join(f'"a{n}"' for n in range(256))
    sclob = ", ".join(f'"s{n}"' for n in range(S_BASE, S_DA2 + 1))
    parts.append(f"#define DFP4_NATIVE_VGPR_CLOBBERS {vclob}\n")
    parts.append(f"#define DFP4_NATIVE_ACC_CLOBBERS {aclob}\n")
    parts.append(f"#define DFP4_NATIVE_SGPR_CLOBBERS {sclob}\n")
    path = os.path.join(here, "gemm_native_asm.inc")
    text = "\n".join(parts)
    if not os.path.exists(path) or open(path).read() != text:
        with open(path, "w") as fh:
            fh.write(text)
    return path


if __name__ == "__main__":
    print(main())
