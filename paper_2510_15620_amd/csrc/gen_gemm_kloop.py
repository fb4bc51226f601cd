#!/usr/bin/env python3
"""Generates gemm_16_kloop.inc: the hand-scheduled K loops of the GEMM tiles.

    python gen_gemm_kloop.py > gemm_16_kloop.inc        (the output is committed too)

The 256x256x64 tile.  4 wavefronts (one per SIMD, so each owns 512 registers), wave grid 2x2, wave tile 128x128 = 8x8
accumulator tiles of v_mfma_f32_16x16x32 kept in 256 AGPRs: the largest wave tile the register file allows, i.e. the
fewest LDS bytes per MFMA.  A slice is 64 deep: 2 steps of 64 MFMAs (16 cycles each, 2048 in all).

What bounds it: power.  On operands that toggle the chip lowers its clock until the energy per flop fits, so time follows
the energy of a slice first and its stalls second.  Measured on f16 normals, 24576 x 24576 x 4096 / 32768 x 4096 x 12288 (a
product alone, no memory traffic at all, reaches 1600-1620 TFLOP/s):
  * 32x32x16 MFMAs, two stages, loads in two bursts of 8: 1228-1252 / 1181-1205 TFLOP/s (1.53 us a slice at 1.59 GHz, pipes 85 %
    busy inside the loop; 74 % down projection);
  * 16x16x32 MFMAs and single loads: 1365-1375 / 1330-1340 (1.38 us at 1.73 GHz, as busy: the same product - to the bit - for
    less energy; alone the two instructions are level, 1590 against 1620);
  * + pairs of rows in the MFMA order (below) and 4 row tiles a group: 1410 / 1340;
  * + a third stage for A, loads spread over three quarters of a slice: 1427 / 1420 (93 % busy at 1.57-1.65 GHz).

Pipeline (t = slice, positions are MFMAs 0..127 of the slice):
  * global memory -> LDS directly (global_load_lds_dwordx4, no staging registers).  Each instruction fills 8 tile rows
    (1 KiB); the XOR swizzle is applied on the source side (lane l fetches the chunk that belongs in slot l % 8 of row l / 8);
  * LDS holds three stages of A and two of B (160 KiB).  Behind the slice's barrier (position PB) the stages of slice t are
    free: B of slice t+2 and then A of slice t+3 are requested, one load every LSTRIDE MFMAs.  Every 3, 4, 5, 7 or 8 was slower: a
    load occupies the CU's address path for 16 cycles, the four waves issue theirs together, and a wave that waits there
    issues no MFMA;
  * the barrier waits for all but the 8 youngest loads (A of slice t+2): B has a whole slice to arrive, A two;
  * LDS -> fragments one step ahead into the other of two register sets, one read every RSTRIDE MFMAs.
Near the end of K the loads re-read the last slice (in bounds, into stages nobody reads), which keeps the slice bodies
free of branches.  The stage offsets are immediates, so the loop is unrolled over 6 slices.

The W fragment is the first MFMA operand, so accumulator tiles come out transposed (a lane owns one row of A).
"""
# ---- register plan (all clobbered) ----
AA, AA2, AB, AB2 = [116, 117], [118, 119], [120, 121], [122, 123]   # LDS address of the lane's first fragment row, per step: A stages
                                                                    # 0 and 1, A stage 2, B columns 0-63, B columns 64-127 of the wave
F = [{"A": [128 + 64 * s + 4 * i for i in range(8)], "B": [160 + 64 * s + 4 * j for j in range(8)]} for s in range(2)]
CLOBBER_V = list(range(116, 124)) + list(range(128, 256))
CLOBBER_S = list(range(20, 30))

STAGE = 32768                           # bytes per LDS stage of one operand
A_STAGES, B_STAGES, PERIOD = 3, 2, 6
TILE_ROWS = 2048                        # 16 rows x 128 B
RSTRIDE, PB, LSTRIDE = 3, 56, 6


def v4(r):
    return f"v[{r}:{r + 3}]"


def acc(i, j):
    """16 x 16 tile (i, j) of the wave: the 32 x 32 block (i / 2, j / 2) is operand acc[i / 2][j / 2] of the kernel, 16 registers, its
    four tiles in the order (0,0), (0,1), (1,0), (1,1)."""
    r = ((i // 2) * 4 + j // 2) * 16 + ((i % 2) * 2 + j % 2) * 4
    return f"a[{r}:{r + 3}]"


def reads(fs, k, t):
    """The 16 fragment reads of step k of slice t into fragment set fs, in the order of their first use."""
    sa, sb = t % A_STAGES, t % B_STAGES
    base, off = (AA2, 0) if sa == 2 else (AA, sa * STAGE)              # a read's immediate offset ends at 64 KiB
    ra = lambda i: f"ds_read_b128 {v4(F[fs]['A'][i])}, v{base[k]} offset:{off + i * TILE_ROWS}"
    rb = lambda j: f"ds_read_b128 {v4(F[fs]['B'][j])}, v{(AB if j < 4 else AB2)[k]} offset:{sb * STAGE + j % 4 * TILE_ROWS}"
    return [ra(0), rb(0), ra(1)] + [rb(j) for j in range(1, 8)] + [ra(i) for i in range(2, 8)]


def mfma(fs, i, j):
    return f'v_mfma_f32_16x16x32_" TY " {acc(i, j)}, {v4(F[fs]["B"][j])}, {v4(F[fs]["A"][i])}, {acc(i, j)}'


def loads(which, stage):
    """8 direct-to-LDS loads of this wave for one operand: M0 = LDS destination (wave base + 1 KiB per instruction + stage),
    source = running base s[20:21] / s[22:23] + the lane's byte offset."""
    base, lds, off = ("s[20:21]", "%[la]", "ga") if which == "A" else ("s[22:23]", "%[lb]", "gb")
    return [f"s_add_u32 m0, {lds}, {stage * STAGE + j * 1024}\\n s_nop 0\\n global_load_lds_dwordx4 %[{off}{j}], {base}"
            for j in range(8)]


def advance(which):
    """Moves one operand's base to the next slice while that stays inside the operand (s25 / s29 = index of the slice the
    base points at, s26 = last slice)."""
    idx, lo, hi = ("s25", "s20", "s21") if which == "A" else ("s29", "s22", "s23")
    return [f"s_cmp_lt_u32 {idx}, s26", "s_cselect_b32 s27, 128, 0", "s_cselect_b32 s28, 1, 0",
            f"s_add_u32 {lo}, {lo}, s27", f"s_addc_u32 {hi}, {hi}, 0", f"s_add_u32 {idx}, {idx}, s28"]


def mfma_order():
    """Two rows of accumulator tiles at a time, column by column, turning at the ends: consecutive MFMAs differ in one operand
    fragment (fewer operand bits toggle; 0.8 % faster than row by row)."""
    out = []
    for p in range(4):
        for n, j in enumerate(range(8) if p % 2 == 0 else range(7, -1, -1)):
            out += [(2 * p + i, j) for i in ((0, 1) if n % 2 == 0 else (1, 0))]
    return out


def slice_body(t):
    behind = {}                                         # position -> what is issued behind that MFMA
    for n, r in enumerate(reads(1, 1, t)):
        behind.setdefault(n * RSTRIDE, []).append(r)
    for n, r in enumerate(reads(0, 0, t + 1)):
        behind.setdefault(64 + n * RSTRIDE, []).append(r)
    # the loads requested behind this slice's barrier, and those of the slice before that reach into this one (they go to the
    # stages that were freed by its barrier)
    for s, shift in ((t, 0), (t - 1, 128)):
        for n, l in enumerate(loads("B", s % B_STAGES) + loads("A", s % A_STAGES)):
            p = PB + 1 + n * LSTRIDE - shift
            if 0 <= p < 128 and (shift == 0 or p < PB):
                behind.setdefault(p, []).append(l)
    assert 15 * RSTRIDE < PB and PB + 1 + 15 * LSTRIDE - 128 < PB
    out = []
    for m in range(128):
        if m in (0, 64):
            out.append("s_waitcnt lgkmcnt(0)")          # the step's fragments; the last was requested 18 MFMAs ago
        if m == PB:
            out += ["s_waitcnt vmcnt(8) lgkmcnt(0)"] + advance("A") + advance("B") + ["s_barrier"]
        out.append(mfma(m // 64, *mfma_order()[m % 64]))
        out += behind.get(m, [])
    return out


def kloop():
    s = []
    for k in range(2):                                  # the steps' addresses differ only in a swizzled chunk bit
        s += [f"v_xor_b32 v{r[k]}, {64 * k}, %[{a}]" for r, a in ((AA, "aa"), (AB, "ab"), (AB2, "ab2"))]
        s += [f"v_add_u32 v{AA2[k]}, {2 * STAGE}, v{AA[k]}"]
    s += ["s_mov_b64 s[20:21], %[pa]", "s_mov_b64 s[22:23], %[pb]", "s_mov_b32 s24, %[nk]", "s_sub_u32 s26, %[nk], 1",
          "s_mov_b32 s25, 0", "s_mov_b32 s29, 0"]
    # ---- prologue: B and A of slices 0 and 1, A of slice 2; the accumulators are cleared while the first of them arrive
    s += loads("B", 0) + advance("B") + loads("A", 0) + advance("A") + loads("B", 1) + loads("A", 1) + advance("A") + loads("A", 2)
    s += [f"v_accvgpr_write_b32 a{r}, 0" for r in range(256)]
    s += ["s_waitcnt vmcnt(24)", "s_barrier"] + reads(0, 0, 0)
    s += ["L_loop_%=:"]
    for t in range(PERIOD):
        s += slice_body(t) + ["s_sub_u32 s24, s24, 1", "s_cmp_eq_u32 s24, 0"]
        s += ["s_cbranch_scc1 L_done_%="] if t + 1 < PERIOD else ["s_cbranch_scc0 L_loop_%="]
    s += ["L_done_%=:", "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_nop 15", "s_nop 15"]   # MFMA results settle before the epilogue reads them
    return s


# ------------------------------------------------------------------------------------------------ small tiles
# K loop of the tiles below 256 x 256 (see gemm_16.hip for when they are used).  Such launches have few tiles per compute
# unit, often less than one, so a slice's time is a chain of latencies: what counts is how many slices of loads are in
# flight and that nothing but the MFMAs and one barrier is left on the chain.
#   * LDS holds a ring of S slices; slice t+S is requested while slice t feeds the MFMAs, so S-1 slices are in flight;
#   * fragments are read one phase ahead into the other of two register sets (a phase is a whole slice, or half of one
#     where the sets would not fit), so a phase's MFMAs start without a wait;
#   * one barrier per slice: behind it slice t+1 has landed for everybody, and everybody has the last fragments of
#     slice t in registers, so its stage may be overwritten.
# The ring is unrolled (stage offsets are immediates).  Loads take their row offsets as inputs, one register per load
# instruction, so rows beyond the matrix are clamped by the caller and edge tiles run the same loop.
S_AA, S_AB, S_F = 24, 28, 32              # first VGPRs: step addresses of A and B, fragments


class Small:
    def __init__(self, name, TM, TN, nla, nlb, bm, bn, S, b_off, ks):
        self.name, self.TM, self.TN, self.nla, self.nlb, self.S, self.ks = name, TM, TN, nla, nlb, S, ks
        self.a_stage, self.b_stage, self.b_off = bm * 128, bn * 128, b_off
        n = TM * TN
        self.aA, self.aB = n, n + 1
        self.gA, self.gB = n + 2, n + 2 + nla
        self.ldsA = n + 2 + nla + nlb
        self.ldsB, self.baseA, self.baseB, self.nk = self.ldsA + 1, self.ldsA + 2, self.ldsA + 3, self.ldsA + 4
        self.set_regs = ks * (TM + TN) * 4
        self.last_v = S_F + 2 * self.set_regs - 1

    def frag(self, st, kk, which, i):
        at = S_F + st * self.set_regs + (kk % self.ks) * (self.TM + self.TN) * 4 + (i if which == "A" else self.TM + i) * 4
        return v4(at)

    def reads(self, st, phase, stage):
        out = []
        for kk in range(phase * self.ks, (phase + 1) * self.ks):
            for i in range(self.TM):
                out.append(f"ds_read_b128 {self.frag(st, kk, 'A', i)}, v{S_AA + kk} offset:{stage * self.a_stage + i * 4096}")
            for j in range(self.TN):
                out.append(f"ds_read_b128 {self.frag(st, kk, 'B', j)}, v{S_AB + kk} offset:{stage * self.b_stage + self.b_off[j]}")
        return out

    def loads(self, stage):
        out = []
        for j in range(self.nla):
            out.append(f"s_add_u32 m0, %{self.ldsA}, {stage * self.a_stage + j * 1024}\\n s_nop 0\\n global_load_lds_dwordx4 %{self.gA + j}, s[20:21]")
        for j in range(self.nlb):
            out.append(f"s_add_u32 m0, %{self.ldsB}, {stage * self.b_stage + j * 1024}\\n s_nop 0\\n global_load_lds_dwordx4 %{self.gB + j}, s[22:23]")
        return out

    def advance(self):
        """Both bases to the next slice while that exists (s25 = slice the bases point at, s26 = last slice): near the end
        the loads re-read the last slice, in bounds, into stages that nobody reads any more."""
        return ["s_cmp_lt_u32 s25, s26", "s_cselect_b32 s27, 128, 0", "s_cselect_b32 s28, 1, 0", "s_add_u32 s20, s20, s27",
                "s_addc_u32 s21, s21, 0", "s_add_u32 s22, s22, s27", "s_addc_u32 s23, s23, 0", "s_add_u32 s25, s25, s28"]

    def mfmas(self, mn, st, phase):
        out = []
        for kk in range(phase * self.ks, (phase + 1) * self.ks):
            for i in range(self.TM):
                for jj in range(self.TN):
                    j = jj if i % 2 == 0 else self.TN - 1 - jj
                    acc = f"%{i * self.TN + j}"
                    out.append(f"{mn} {acc}, {self.frag(st, kk, 'B', j)}, {self.frag(st, kk, 'A', i)}, {acc}")
        return out

    def text(self, mn):
        L, S, np_ = self.nla + self.nlb, self.S, 4 // self.ks
        s = []
        for k in range(4):
            s += [f"v_xor_b32 v{S_AA + k}, {32 * k}, %{self.aA}", f"v_xor_b32 v{S_AB + k}, {32 * k}, %{self.aB}"]
        s += [f"s_mov_b64 s[20:21], %{self.baseA}", f"s_mov_b64 s[22:23], %{self.baseB}", f"s_mov_b32 s24, %{self.nk}",
              f"s_sub_u32 s26, %{self.nk}, 1", "s_mov_b32 s25, 0"]
        for t in range(S - 1):
            s += self.loads(t) + self.advance()
        s += [f"s_waitcnt vmcnt({(S - 2) * L})", "s_barrier"]
        s += self.reads(0, 0, 0) + self.loads(S - 1) + self.advance()
        s += ["L_loop_%=:"]
        # one turn of the ring; with an odd number of phases per turn the register sets would not alternate, so two turns
        turns = 1 if (S * np_) % 2 == 0 else 2
        st = 0
        for t in range(S * turns):
            p = t % S
            for ph in range(np_):
                last = ph == np_ - 1
                s += [f"s_waitcnt vmcnt({(S - 2) * L}) lgkmcnt(0)", "s_barrier"] if last else ["s_waitcnt lgkmcnt(0)"]
                nxt = self.reads(1 - st, 0, (p + 1) % S) if last else self.reads(1 - st, ph + 1, p)
                mf = self.mfmas(mn, st, ph)
                ld = self.loads(p) if last else []
                # fragment reads first (they are on the next phase's chain), two behind every MFMA; loads behind them
                k = 0
                for m in mf:
                    s.append(m)
                    take = max(2, -(-len(nxt) // max(1, len(mf) // 2)))
                    s += nxt[k:k + take]
                    if k >= len(nxt) and ld:
                        n = -(-len(ld) // max(1, len(mf) // 2))
                        s += ld[:n]
                        ld = ld[n:]
                    k += take
                s += nxt[k:] + ld
                if last:
                    s += self.advance()
                st = 1 - st
            s += ["s_sub_u32 s24, s24, 1", "s_cmp_eq_u32 s24, 0"]
            s += ["s_cbranch_scc1 L_done_%="] if t + 1 < S * turns else ["s_cbranch_scc0 L_loop_%="]
        s += ["L_done_%=:", "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_nop 15", "s_nop 15"]
        return s

    def emit(self):
        for tname, mn in (("F16", "v_mfma_f32_32x32x16_f16"), ("BF16", "v_mfma_f32_32x32x16_bf16")):
            emit(f"PRISM_KLOOP_{tname}_{self.name}", self.text(mn))
        regs = ", ".join(f'"v{r}"' for r in range(S_AA, self.last_v + 1)) + ", " + ", ".join(f'"s{r}"' for r in range(20, 29))
        print(f"#define PRISM_KLOOP_CLOBBERS_{self.name} {regs}, \"scc\", \"memory\"")
        print()


#   name (tile, ring depth): accumulator tiles per wave, loads per wave and slice, tile, ring depth, B fragment offsets,
#   k-steps per register set
SMALL = [
    Small("32x32_8", 1, 1, 4, 4, 32, 32, 8, [0], 4),
    Small("64x32_6", 1, 1, 4, 2, 64, 32, 6, [0], 4),
    Small("32x64_4", 1, 2, 4, 8, 32, 64, 4, [0, 4096], 4),
    Small("64x64_5", 1, 2, 4, 4, 64, 64, 5, [0, 4096], 4),
    Small("128x64_3", 1, 2, 4, 2, 128, 64, 3, [0, 4096], 4),
    Small("128x128_3_PLAIN", 2, 2, 4, 4, 128, 128, 3, [0, 4096], 2),
    Small("128x128_3_SWIGLU", 2, 2, 4, 4, 128, 128, 3, [0, 8192], 2),
    Small("128x128_2_PLAIN", 2, 2, 4, 4, 128, 128, 2, [0, 4096], 2),
    Small("128x128_2_SWIGLU", 2, 2, 4, 4, 128, 128, 2, [0, 8192], 2),
    # q/k/v projection: a wave owns the 128 columns of one head
    Small("64x128_3_HEAD", 1, 4, 4, 8, 64, 128, 3, [0, 4096, 8192, 12288], 2),
    Small("128x128_3_HEAD", 1, 4, 4, 4, 128, 128, 3, [0, 4096, 8192, 12288], 2),
    Small("128x128_2_HEAD", 1, 4, 4, 4, 128, 128, 2, [0, 4096, 8192, 12288], 2),
]


def emit(name, lines):
    print(f"#define {name} \\")
    for l in lines:
        print(f'  "{l}\\n" \\')
    print('  ""')
    print()


def main():
    print("// Generated by gen_gemm_kloop.py - do not edit.  See that file for the schedule.")
    print("// PRISM_KLOOP_256(TY), TY = \"f16\" or \"bf16\": accumulators a[0:255] (32 x 32 block (i, j) of the wave in a[(4i+j)*16 : +15]);")
    print("// aa / ab / ab2 LDS byte address of the lane's first fragment row of A, of B columns 0-63 and 64-127 (step 0, stage 0);")
    print("// ga0..7 / gb0..7 byte offset into A / W of the chunk this lane fetches in each of its wave's load instructions; la / lb")
    print("// LDS byte address of the first row the first of them fills (stage 0, uniform); pa / pb base of A / W; nk number of slices.")
    print("// PRISM_KLOOP_*: accumulators acc[i][j] first (AGPRs), then the same values by position (see class Small).")
    print()
    emit("PRISM_KLOOP_256(TY)", kloop())
    regs = ", ".join(f'"v{r}"' for r in CLOBBER_V) + ", " + ", ".join(f'"s{r}"' for r in CLOBBER_S)
    for c in SMALL:
        c.emit()
    # m0 (written before every direct-to-LDS load) is not listed: the compiler reserves it, sets it right before each of
    # its own uses and never keeps a value in it across a statement; hipcc diagnoses it in a clobber list
    print(f"#define PRISM_KLOOP_256_CLOBBERS {regs}, \"scc\", \"memory\"")


if __name__ == "__main__":
    main()
