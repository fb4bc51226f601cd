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
import math

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
    r = (i * 8 + j) * 4
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


def load_group(which, n, lds_off, m0_at=0):
    """Direct-to-LDS loads 0 .. n - 1 of this wave for one operand: M0 = LDS destination (wave base + stage + 4 KiB per four
    loads, set before loads m0_at, 4, 8, ..), source = running base s[20:21] / s[22:23] + the lane's byte offset; the instruction's
    offset is added to both (the lane's comes without it)."""
    base, lds, off = ("s[20:21]", "%[la]", "ga") if which == "A" else ("s[22:23]", "%[lb]", "gb")
    m0 = lambda j: f"s_add_u32 m0, {lds}, {lds_off + j // 4 * 4096}\\n s_nop 0\\n " if j % 4 == 0 or j == m0_at else ""
    return [f"{m0(j)}global_load_lds_dwordx4 %[{off}{j}], {base} offset:{j % 4 * 1024}" for j in range(n)]


def loads(which, stage):
    return load_group(which, 8, stage * STAGE)


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
# unit, often less than one, so a slice's time is a chain of latencies and of what its few waves issue: what counts is how
# many slices of loads are in flight, that the MFMAs start without a wait and that little but them is left to issue.
#   * 16x16x32 MFMAs, as in the large tile: the waves of a small tile then have 2 to 32 independent accumulators instead of
#     one or two, and a tile can be cut over four waves down to 16 x 16 each;
#   * LDS holds a ring of S slices;
#   * fragments are read RA steps (of 32 k) ahead.  RA = 1: the barrier stands in the middle of a slice, when its last
#     fragments have landed: its stage is free, S - 1 slices are in flight.  RA = 2, 4 for waves whose step is too short to
#     cover an LDS read: RA - 1 steps of reads stay outstanding at the barrier, at the start of a slice, so the stage freed
#     is the slice's before, and S - 1 - RA / 2 slices are in flight;
#   * a launch of a few rows streams its weights from memory, and the slices in flight are what it has to cover that latency
#     with: 7 of 32 x 32, 5 of 64 x 32, 3 of 32 x 64.  Fragments four steps ahead in a ring of 8, or two steps ahead in rings of 6 and 4,
#     left 5, 4 and 2 and were level or faster only on operands that stay in the caches.  us, weights from memory, those rings -> these:
#     1 x 4096 x 12288 29.7 -> 24.1, 33 x 2560 x 9728 22.3 -> 18.5, 6 x 1024 x 3072 8.6 -> 7.4 (32 x 32); 100 x 4096 x 12288 38.0 ->
#     37.0, 391 x 1024 x 3072 10.5 -> 9.8 (64 x 32); with SwiGLU 1 x 6144 x 1024 8.0 -> 7.2, 1 x 24576 x 4096 40.9 -> 39.1 (32 x 64; two waves
#     with the same ring: 6.7 and 38.8, but 32 x 19456 x 2560 28.2 instead of 27.4, two tiles on a few units being what it waits for);
#   * the tiles of 128 rows have a second, deeper ring for launches that give a compute unit one tile at most, where the LDS that
#     a second workgroup would use is free (gemm_16.hip: deep_ring).  Not the smaller tiles: rings of 8 to 18 slices, fragments 4 to 8 steps
#     ahead or not, change their times by under 3 % (they stand at some 25 bytes per cycle and unit, whatever is in flight);
#   * loads are spread over the slice; four of them share one M0, their offsets shift source and destination alike.
# The ring is unrolled (stage offsets are immediates).  Loads take their row offsets as inputs, one register per load
# instruction, so rows beyond the matrix are clamped by the caller and edge tiles run the same loop.
# Against 32x32x16 loops with the same tiles, us, operands that stay in the caches: 777 x 6144 x 1024 with SwiGLU 17.4 -> 15.4
# (128 x 128, two stages), 3699 x 1024 x 3072 30.9 -> 29.1 (128 x 128 deep), 391 x 4096 x 1024 with heads 10.8 -> 9.4 (64 x 128 on four
# waves instead of two), 6 x 1024 x 3072 7.2 -> 5.3 (32 x 32 on four waves instead of one), 391 x 1024 x 3072 8.9 -> 8.7 (64 x 32;
# four waves are no faster); weights from memory: the last two 7.7 -> 7.4 and 9.9 -> 9.8.
FIRST_V = 24                            # first VGPR: step addresses, then fragments


class Small:
    def __init__(self, name, bm, bn, wm, wn, S, RA, sets):
        nw = wm * wn
        self.name, self.S, self.RA, self.sets, self.ahead = name, S, RA, sets, RA // 2
        self.TM, self.TN = bm // wm // 16, bn // wn // 16
        self.nla, self.nlb = bm // 8 // nw, bn // 8 // nw                 # loads of a wave and slice
        self.L, self.R, self.NS = self.nla + self.nlb, self.TM + self.TN, self.TM * self.TN
        self.a_stage, self.b_stage = bm * 128, bn * 128
        self.high = S * max(bm, bn) * 128 > 65536                         # a read's immediate offset ends at 64 KiB
        self.f0 = FIRST_V + (12 if self.high else 8)
        self.last_v = self.f0 + sets * self.R * 4 - 1
        assert (RA - 1) * self.R <= 15 and (S - 1) * self.L <= 63         # what the wait counters can hold
        assert sets > RA and (RA == 1 or (RA % 2 == 0 and S >= self.ahead + 2)) and S * (bm + bn) * 128 <= 163840

    def addr(self, which, k, high):
        return FIRST_V + {"A": 0, "B": 2, "B2": 4}[which] + k + (6 if high else 0)

    def frag(self, u, which, i):
        return v4(self.f0 + (u % self.sets) * self.R * 4 + (i if which == "A" else self.TM + i) * 4)

    def reads(self, u):
        """The fragment reads of step u (slice u / 2): the lower half of the wave's columns through one address, the upper through another
        (SwiGLU's upper half are the up rows)."""
        t, k, half = u // 2, u % 2, max(self.TN // 2, 1)

        def rd(which, i):
            off = t % self.S * self.a_stage + i * TILE_ROWS if which == "A" else t % self.S * self.b_stage + i % half * TILE_ROWS
            r = which if which == "A" or i < half else "B2"
            return f"ds_read_b128 {self.frag(u, which, i)}, v{self.addr(r, k, off >= 65536)} offset:{off % 65536}"
        return [rd("A", 0)] + [rd("B", j) for j in range(self.TN)] + [rd("A", i) for i in range(1, self.TM)]

    def loads(self, stage, first=0):
        """The loads of one slice from number `first` on."""
        out = load_group("A", self.nla, stage * self.a_stage) + load_group("B", self.nlb, stage * self.b_stage)
        which, n, at = ("A", first, stage * self.a_stage) if first < self.nla else ("B", first - self.nla, stage * self.b_stage)
        return load_group(which, n + 1, at, n)[n:] + out[first + 1:] if first else out

    def advance(self, exists):
        """Both bases to the next slice if that exists: near the end the loads re-read the last slice, in bounds, into stages
        that nobody reads any more."""
        return [exists, "s_cselect_b32 s25, 128, 0", "s_add_u32 s20, s20, s25", "s_addc_u32 s21, s21, 0", "s_add_u32 s22, s22, s25",
                "s_addc_u32 s23, s23, 0"]

    def text(self):
        S, RA, NS, L, N = self.S, self.RA, self.NS, self.L, 2 * self.NS
        s = []
        for k in range(2):
            for which, a in (("A", "aa"), ("B", "ab"), ("B2", "ab2")):
                s.append(f"v_xor_b32 v{self.addr(which, k, False)}, {64 * k}, %[{a}]")
                if self.high:
                    s.append(f"v_add_u32 v{self.addr(which, k, True)}, 65536, v{self.addr(which, k, False)}")
        s += ["s_mov_b64 s[20:21], %[pa]", "s_mov_b64 s[22:23], %[pb]", "s_sub_u32 s24, %[nk], 1"]    # s24: slices after this one
        n_pro = S if RA == 1 else S - 1
        for t in range(n_pro):
            s += self.loads(t) + (self.advance(f"s_cmp_gt_u32 s24, {t}") if t + 1 < n_pro else [])
        s += [f"v_accvgpr_write_b32 a{r}, 0" for r in range((self.TM * self.TN + 3) // 4 * 16)]
        s += [f"s_waitcnt vmcnt({(n_pro - max(self.ahead, 1)) * L})", "s_barrier"]
        for u in range(RA):
            s += self.reads(u)
        order = [(i, j if i % 2 == 0 else self.TN - 1 - j) for i in range(self.TM) for j in range(self.TN)]
        bar = NS if RA == 1 else 0                               # the barrier's place
        landed = (S - 2 - self.ahead) * L
        outstanding = f"lgkmcnt({(RA - 1) * self.R})"
        period = math.lcm(S, self.sets // math.gcd(2, self.sets))
        s += ["L_loop_%=:"]
        for t in range(period):
            behind = {}
            for h in range(2):
                for n, r in enumerate(self.reads(2 * t + h + RA)):
                    behind.setdefault(h * NS + n * NS // self.R, []).append(r)
            # loads requested behind this slice's barrier, and, where that stands in the middle, the slice before's that reach into
            # this one: the first turn repeats the youngest slice's there, so the first of them sets M0 itself
            at = [bar + n * N // L for n in range(L)]
            here = [n for n in range(L) if at[n] < N]
            for n in here:
                behind.setdefault(at[n], []).append(self.loads((t if RA == 1 else t - 1) % S)[n])
            tail = [n for n in range(L) if at[n] >= N]
            for n in tail:
                assert at[n] - N < bar
                behind.setdefault(at[n] - N, []).append(self.loads((t - 1) % S, tail[0])[n - tail[0]])
            for m in range(N):
                if m == bar:
                    s += [f"s_waitcnt vmcnt({landed}) {outstanding}"] + self.advance(f"s_cmp_ge_u32 s24, {n_pro}") + ["s_barrier"]
                elif m % NS == 0:
                    s += [f"s_waitcnt {outstanding}"]
                (i, j), u = order[m % NS], 2 * t + m // NS
                r = (i * self.TN + j) * 4
                s.append(f'v_mfma_f32_16x16x32_" TY " a[{r}:{r + 3}], {self.frag(u, "B", j)}, {self.frag(u, "A", i)}, a[{r}:{r + 3}]')
                s += behind.get(m, [])
            s += ["s_sub_u32 s24, s24, 1"] + (["s_cbranch_scc1 L_done_%="] if t + 1 < period else ["s_cbranch_scc0 L_loop_%="])
        s += ["L_done_%=:", "s_waitcnt vmcnt(0) lgkmcnt(0)", "s_nop 15", "s_nop 15"]
        return s

    def emit(self):
        emit(f"PRISM_KLOOP_{self.name}(TY)", self.text())
        regs = ", ".join(f'"v{r}"' for r in range(FIRST_V, self.last_v + 1)) + ", " + ", ".join(f'"s{r}"' for r in range(20, 26))
        print(f"#define PRISM_KLOOP_CLOBBERS_{self.name} {regs}, \"scc\", \"memory\"")
        print()


#   name (tile_stages), tile, wave grid, ring depth, steps read ahead, fragment sets
SMALL = [
    Small("32x32_9", 32, 32, 2, 2, 9, 2, 4),
    Small("64x32_7", 64, 32, 2, 1, 7, 2, 4),
    Small("32x64_4", 32, 64, 1, 1, 4, 1, 2),
    Small("64x64_5", 64, 64, 2, 2, 5, 1, 2),
    Small("128x64_3", 128, 64, 4, 1, 3, 1, 2),
    Small("128x128_4", 128, 128, 2, 2, 4, 2, 4),
    Small("128x128_2", 128, 128, 2, 2, 2, 1, 2),
    # the ring over nearly a whole compute unit's LDS, for launches of at most one tile per unit
    Small("128x64_6", 128, 64, 4, 1, 6, 1, 2),
    Small("128x128_5", 128, 128, 2, 2, 5, 1, 2),
    # q/k/v projection: a wave owns the 128 columns of one head
    Small("64x128_6_HEAD", 64, 128, 4, 1, 6, 1, 2),
    Small("128x128_5_HEAD", 128, 128, 4, 1, 5, 1, 2),
    Small("64x128_3_HEAD", 64, 128, 4, 1, 3, 1, 2),
    Small("128x128_3_HEAD", 128, 128, 4, 1, 3, 1, 2),
    Small("128x128_2_HEAD", 128, 128, 4, 1, 2, 1, 2),
]


def emit(name, lines):
    print(f"#define {name} \\")
    for l in lines:
        print(f'  "{l}\\n" \\')
    print('  ""')
    print()


def main():
    print("// Generated by gen_gemm_kloop.py - do not edit.  See that file for the schedule.")
    print("// PRISM_KLOOP_<tile>(TY), TY = \"f16\" or \"bf16\": accumulators a[0:...], tile (i, j) of 16 x 16 in the four from 4 (TN i + j) on;")
    print("// aa / ab / ab2 LDS byte address of the lane's first fragment row of A, of the lower and of the upper half of the wave's B columns")
    print("// (step 0, stage 0); ga / gb byte offset from pa / pb of the chunk this lane fetches in each of its wave's load instructions,")
    print("// less 1024 (j % 4); la / lb LDS byte address of the first row the first of them fills (stage 0, uniform); nk number of slices.")
    print()
    emit("PRISM_KLOOP_256(TY)", kloop())
    regs = ", ".join(f'"v{r}"' for r in CLOBBER_V) + ", " + ", ".join(f'"s{r}"' for r in CLOBBER_S)
    for c in SMALL:
        c.emit()
    # m0 (written before the direct-to-LDS loads) is not listed: the compiler reserves it, sets it right before each of
    # its own uses and never keeps a value in it across a statement; hipcc diagnoses it in a clobber list
    print(f"#define PRISM_KLOOP_CLOBBERS_256 {regs}, \"scc\", \"memory\"")


if __name__ == "__main__":
    main()
