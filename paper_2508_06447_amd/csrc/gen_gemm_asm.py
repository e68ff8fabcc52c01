#!/usr/bin/env python3
"""Writes gemm_bf16_mainloops.inc: the k-loops of the bf16 projection kernels ("QKV Generation", output projection
and "FFN" of Fig. 2) as gfx950 assembly inside C++ device functions, one per wave-tile shape.  csrc/gemm.hip
includes the file; its C++ part computes the operands and runs the epilogues on the accumulators the functions
return.  Run `python gen_gemm_asm.py` after changing this file (an argument names another output directory); the .inc is
committed and tests/test_generated_sources.py checks that it is current.

Shape of a workgroup: 4 waves, one per SIMD, arranged 2 (features) x 2 (tokens); a wave owns 32 TW x 32 TA outputs (for
SwiGLU: of each of the NW = 2 weight matrices), 128 x 128 in the large tiles, as 16 x 16 MFMA tiles, so that each fragment read
from LDS feeds eight MFMAs.  The 64 accumulators fill the accumulation registers (they are the asm statement's outputs);
fragments are double-buffered in v0..; a lone wave per SIMD means the order of matrix, LDS and tile-load instructions in
the wave is the schedule, so it is written out here.

Why v_mfma_f32_16x16x32_bf16: the loop runs against the power limit, and per flop the 16 x 16 x 32 instruction reads and writes half the
accumulator bytes of the 32 x 32 x 16 one.  Normal operands from registers, all CUs, nothing else in the loop: 32 x 32 x 16
1840 TFLOP/s, 16 x 16 x 32 2080; consecutive MFMAs that change both operands 2 to 3 % less.  So they come in pairs that share the weight
fragment, and the token fragments are walked back and forth.

k-loop: k-tiles of 64 (tile rows of 128 bytes, 16-byte chunks XOR-swizzled as in gemm.hip), operand tiles global -> LDS directly, into
rings: three weight tiles and two activation tiles (all 160 KB of a CU; three activation tiles where they have 128 rows).  Per k-tile: two
k-steps of 4*TW*TA*NW MFMAs; the fragments of a step are read beside the MFMAs of the step before, also across k-tiles.  The one barrier of
a k-tile sits between its k-steps, when every wave holds the second step's fragments and its own part of the next tile has landed; from
there on the slots just read are refilled.  What bounds the loop below the power limit is how long those tile loads have to arrive: issued in one
burst right behind the barrier they back the wave's instruction issue up behind the memory pipeline, spread out the last of them come late.
With two slots for each operand (loads over three quarters of the way to the barrier that waits for them) zero operands, which
do not reach the power limit, ran at 1440 (8192 x 4096 from 14336) and 1710 TFLOP/s (8192^3); with the third weight slot 1870 and 2080.  So
the activation tile goes first, and the weight tile behind it has until the barrier after the next.  Normal operands, two -> three slots (us):
down projection 4096 x 4096 from 14336 353 -> 319, 9856 rows 864 -> 823, 12288 x 3584 from 18944 1314 -> 1205; SwiGLU 4096 x 14336 from 4096 663
-> 643; 8192^3 731 -> 707.  (Launches of less than a round with short rows lose 2 %: Query + Value of 2000 rows 73.5 -> 75, 85 -> 80 with what the 16 x 16 x 32
instruction gives.)  Products of one k-tile leave the rings alone.  The slots are
immediate offsets and the loop six k-tiles long; one k-tile with the slots in registers takes four vector instructions per k-tile and is 1 % slower.
"""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gen_attn_asm import Ins, vr, sr, V, S, valu, salu, nop, label, branch, raw, fix_hazards, weight   # noqa: E402

RING_W = 3                                                     # weight tiles in LDS
A_TO, W_TO = 0.75, 1.9                                         # k-steps behind the barrier over which the activation, then the weight loads go
FIRST_TO = 0.9                                                 # part of the first k-step over which the loads of the third tiles go
READS_TO = 0.95                                                # part of a k-step over which the fragment reads go
N_ACC_IN_VGPRS = 16                                            # accumulators of 4 registers
S_KPW, S_KPW2, S_KPA, S_CNT, S_LSTW, S_LSTA, S_TMP = 40, 42, 44, 46, 47, 48, 49
FIRST_S, LAST_S = 40, 49


class Shape:
    def __init__(self, TW, TA, NW, resid=False):
        self.TW, self.TA, self.NW = TW, TA, NW
        # resid: out = a . w^T + R.  The wave's part of the residual tile is loaded as MFMA B fragments (lane (token, q)
        # takes features 8q .. 8q+7 of each group of 32 output features: 16-byte loads) and added to the
        # accumulators with two MFMAs per fragment whose A operand is a slice of the identity (row f of the 16-row tile p of the group
        # has its one at k = f + 16p): acc += I . R, exact, no vector ALU work, and the epilogue is the plain one.  The fragments come
        # 64 tokens at a time: requested in the prologue and added behind the first k-tile, then, for 128 tokens, requested there and
        # added behind the second.
        self.resid = resid
        self.NWF, self.NAF = 2 * NW * TW, 2 * TA               # fragments per k-step
        n = 4 * (self.NWF + self.NAF)
        self.FRAG = [0, n]                                     # two fragment buffers: W frags then A frags
        self.WADR = 2 * n                                      # [ks][slot >> 1] LDS addresses of the W fragments
        self.AADR = self.WADR + 4                              # [ks] of the A fragments
        self.WOFS = self.AADR + 2                              # lane offsets of the tile loads: <= 8 W, <= 8 A
        self.AOFS = self.WOFS + 8
        self.TMPV = self.AOFS + 8
        self.BN = 32 * TW * 2                                  # features per matrix in a workgroup tile
        self.WROWS = self.BN * NW
        self.AROWS = 32 * TA * 2
        self.RING_A = 2 if TA == 4 else 3
        self.period = RING_W * self.RING_A if self.RING_A != RING_W else RING_W        # k-tiles until the slots repeat
        self.NLW = self.WROWS // 32                            # wave-loads per wave and k-tile: weights, then activations
        self.NLD = (self.WROWS + self.AROWS) // 32
        self.NLA = self.NLD - self.NLW
        assert self.WROWS == 256 and self.RING_A * self.AROWS <= 512 and self.NLW <= 8 and self.NLA <= 8
        self.ROFS = self.TMPV + 1                              # byte offsets of the lane's residual rows
        self.IDENT = (self.ROFS + self.NAF + 2) & ~1           # two identity slices, 4 registers each (ROFS + NAF stays spare)
        self.RES = self.IDENT + 8                              # residual fragments of four 16-token tiles, 4 registers each
        self.LAST_V = self.RES + 16 * TW - 1 if resid else self.TMPV
        assert self.LAST_V < 244
        self.name = f"{TW}_{TA}_{NW}" + ("_resid" if resid else "")

    def acc(self, w, i, j):
        return f"%[c{(w * 2 * self.TW + i) * self.NAF + j}]"

    def mfma_pair(self, buf, w, i, j0, j1, zero):
        wf = self.FRAG[buf] + 4 * (w * 2 * self.TW + i)
        text, r, wr = [], vr(wf, 4), []
        for j in (j0, j1):
            af, c = self.FRAG[buf] + 4 * (self.NWF + j), self.acc(w, i, j)
            text.append(f"v_mfma_f32_16x16x32_bf16 {c}, {V(wf, 4)}, {V(af, 4)}, {'0' if zero else c}")
            r, wr = r + vr(af, 4) + ([] if zero else [c]), wr + [c]
        return Ins("\\n".join(text), "mfma", r=r, w=wr)

    def res_frag(self, j, g, base):
        return base + 4 * ((j & 3) * self.TW + g)

    def residual_loads(self, batch, base):
        return [Ins(f"global_load_dwordx4 {V(self.res_frag(j, g, base), 4)}, {V(self.ROFS + j)}, %[rbase] offset:{g * 64}", "vmem",
                    r=vr(self.ROFS + j), w=vr(self.res_frag(j, g, base), 4))
                for j in range(4 * batch, 4 * batch + 4) for g in range(self.TW)]

    def residual_mfmas(self, batch, base):
        out = []
        for p in range(2):                                     # a group's two accumulators
            for g in range(self.TW):
                for j in range(4 * batch, 4 * batch + 4):
                    c, a, b = self.acc(0, 2 * g + p, j), self.IDENT + 4 * p, self.res_frag(j, g, base)
                    out.append(Ins(f"v_mfma_f32_16x16x32_bf16 {c}, {V(a, 4)}, {V(b, 4)}, {c}", "mfma",
                                   r=vr(a, 4) + vr(b, 4) + [c], w=[c]))
        return out

    def frag_reads(self, buf, t, ks):
        """Fragments of k-step ks of k-tile t."""
        ws, as_ = t % RING_W, t % self.RING_A
        wadr = self.WADR + 2 * ks + (ws >> 1)
        out = []
        for w in range(self.NW):
            for i in range(2 * self.TW):
                d = self.FRAG[buf] + 4 * (w * 2 * self.TW + i)
                off = ((ws & 1) * self.WROWS + w * self.BN + i * 16) * 128
                out.append(Ins(f"ds_read_b128 {V(d, 4)}, {V(wadr)} offset:{off}", "lds", r=vr(wadr), w=vr(d, 4)))
        for j in range(self.NAF):
            d = self.FRAG[buf] + 4 * (self.NWF + j)
            off = (as_ * self.AROWS + j * 16) * 128
            out.append(Ins(f"ds_read_b128 {V(d, 4)}, {V(self.AADR + ks)} offset:{off}", "lds", r=vr(self.AADR + ks), w=vr(d, 4)))
        return out

    def loads(self, t, weights):
        """The wave's wave-loads of the weight or activation tile t, at the pending pointers; then the pointers move on (they stay on the
        last k-tile once it is reached: later loads re-read it into a slot nobody reads).  Lists of instructions that stay together."""
        out = []
        if weights:
            base, n, ofs, lst, ptrs = t % RING_W * self.WROWS * 128, self.NLW, self.WOFS, S_LSTW, [S_KPW, S_KPW2][:self.NW]
        else:
            base, n, ofs, lst, ptrs = (RING_W * self.WROWS + t % self.RING_A * self.AROWS) * 128, self.NLA, self.AOFS, S_LSTA, [S_KPA]
        for i in range(n):
            p = ptrs[i * 32 // self.BN] if weights else ptrs[0]
            out.append([salu(f"s_add_u32 m0, %[ldsw], {base + i * 4096}", w=["m0", "scc"]),
                        Ins(f"global_load_lds_dwordx4 {V(ofs + i)}, {S(p, 2)}", "vmem", r=vr(ofs + i) + ["m0"] + sr(p, 2))])
        out.append([salu(f"s_sub_u32 {S(lst)}, {S(lst)}, 1", r=sr(lst), w=sr(lst) + ["scc"]),
                    salu(f"s_cmp_gt_i32 {S(lst)}, 0", r=sr(lst), w=["scc"]),
                    salu(f"s_cselect_b32 {S(S_TMP)}, 128, 0", r=["scc"], w=sr(S_TMP))])
        for p in ptrs:
            out.append([salu(f"s_add_u32 {S(p)}, {S(p)}, {S(S_TMP)}", r=sr(p) + sr(S_TMP), w=sr(p) + ["scc"]),
                        salu(f"s_addc_u32 {S(p + 1)}, {S(p + 1)}, 0", r=sr(p + 1) + ["scc"], w=sr(p + 1) + ["scc"])])
        return out

    def refill(self, t):
        """What goes out behind the barrier of k-tile t, as (k-steps behind it, instructions)."""
        return self.timed((self.loads(t + self.RING_A, False), 0, A_TO), (self.loads(t + RING_W, True), A_TO, W_TO))

    def timed(self, *parts):
        """(loads, from, to): as (k-steps, instructions)."""
        pair = 1.0 / (self.NW * 2 * self.TW * self.TA)         # m0 is written an MFMA pair ahead of its load, which saves a wait state
        out, last = [], 0
        for xs, lo, hi in parts:
            for k, x in enumerate(xs):
                at = max(last, lo + (hi - lo) * k / len(xs))   # (and never before the load ahead of it)
                last = at + pair if x[-1].kind == "vmem" else at
                out += [(at, x[:1]), (last, x[1:])] if x[-1].kind == "vmem" else [(at, x)]
        return out

    @staticmethod
    def deal(mf, reads, fills):
        """The fragment reads spread evenly, and the fills (part of the step, instructions), behind the MFMA pairs of a step."""
        behind = [[] for _ in mf]
        for k, x in enumerate(reads):
            behind[int(READS_TO * k / len(reads) * len(mf))].append(x)
        for at, xs in fills:
            behind[min(int(at * len(mf) + 1e-9), len(mf) - 1)] += xs
        return [x for m, xs in zip(mf, behind) for x in [m] + xs]

    def pairs(self, buf, zero):
        """The MFMAs of a k-step from fragment buffer buf."""
        rows = [(w, i) for w in range(self.NW) for i in range(2 * self.TW)]
        order = []
        for n, (w, i) in enumerate(rows):                      # token fragments back and forth
            js = list(range(self.NAF))[::-1 if n & 1 else 1]
            order += [(w, i, js[k], js[k + 1]) for k in range(0, self.NAF, 2)]
        return [self.mfma_pair(buf, *o, zero) for o in order]

    def k_tile(self, t, first, in_flight=None):
        """k-tile t; the fragments of its k-step 0 are in buffer 0 (already requested).  in_flight: loads that may be on their way at its barrier."""
        if first:                                              # the last tiles of the rings that the prologue has left out
            carry = self.timed(((self.loads(2, False) if self.RING_A == 3 else []) + self.loads(2, True), 0, FIRST_TO))
        else:
            carry = [(at - 1, x) for at, x in self.refill(t + self.period - 1) if at >= 1]
        if in_flight is None:
            in_flight = self.NLW + (self.NLA if self.RING_A == 3 else 0)
        seq = [raw("s_waitcnt lgkmcnt(0)", "wait")]
        seq += self.deal(self.pairs(0, first), self.frag_reads(1, t, 1), carry)
        seq += [raw(f"s_waitcnt vmcnt({in_flight}) lgkmcnt(0)", "wait"), raw("s_barrier", "barrier")]
        seq += self.deal(self.pairs(1, False), self.frag_reads(0, t + 1, 0), [(at, x) for at, x in self.refill(t) if at < 1])
        return seq

    def residual_setup(self):
        """Byte offsets of the lane's residual rows: row = min(rrow0 + 16 j, alim) of the workgroup tile."""
        out = []
        for j in range(self.NAF):
            out += [valu(f"v_add_u32 {V(self.TMPV)}, {16 * j}, %[rrow0]", w=vr(self.TMPV)),
                    valu(f"v_min_i32 {V(self.TMPV)}, %[alim], {V(self.TMPV)}", r=vr(self.TMPV), w=vr(self.TMPV)),
                    valu(f"v_mad_u32_u24 {V(self.ROFS + j)}, {V(self.TMPV)}, %[rstride], %[rcol0]", r=vr(self.TMPV), w=vr(self.ROFS + j))]
        return out

    def identity(self):
        """Identity slices: t = f + 16p - 8q with f = rrow0 & 15 and q = bits 4 and 5 of rcol0; the lane's one is
        bf16 element t of its 8 (if 0 <= t < 8): dword t >> 1, upper half if t is odd."""
        out = []
        e = out.append
        t, val, idx = self.TMPV, self.ROFS + self.NAF, self.TMPV         # ROFS + NAF is a spare register below IDENT
        for p in range(2):
            e(valu(f"v_and_b32 {V(t)}, 15, %[rrow0]", w=vr(t)))
            e(valu(f"v_bfe_u32 {V(val)}, %[rcol0], 4, 2", w=vr(val)))
            e(valu(f"v_lshlrev_b32 {V(val)}, 3, {V(val)}", r=vr(val), w=vr(val)))
            e(valu(f"v_sub_u32 {V(t)}, {V(t)}, {V(val)}", r=vr(t) + vr(val), w=vr(t)))
            e(valu(f"v_add_u32 {V(t)}, {16 * p}, {V(t)}", r=vr(t), w=vr(t)))
            sh = self.IDENT + 7                            # free until the last select of p = 1 writes it
            e(valu(f"v_and_b32 {V(sh)}, 1, {V(t)}", r=vr(t), w=vr(sh)))
            e(valu(f"v_lshlrev_b32 {V(sh)}, 4, {V(sh)}", r=vr(sh), w=vr(sh)))
            e(valu(f"v_mov_b32 {V(val)}, 0x3f80", w=vr(val)))                  # bf16 1.0
            e(valu(f"v_lshlrev_b32 {V(val)}, {V(sh)}, {V(val)}", r=vr(sh) + vr(val), w=vr(val)))
            e(valu(f"v_ashrrev_i32 {V(idx)}, 1, {V(t)}", r=vr(t), w=vr(idx)))
            for dw in range(4):
                e(valu(f"v_cmp_eq_u32 vcc, {dw}, {V(idx)}", r=vr(idx), w=["vcc"], kind="vcmp"))
                e(valu(f"v_cndmask_b32 {V(self.IDENT + 4 * p + dw)}, 0, {V(val)}, vcc", r=vr(val) + ["vcc"], w=vr(self.IDENT + 4 * p + dw)))
        return out

    def only_k_tile(self):
        """The whole product where it has one k-tile, whose loads have been issued: no rings, nothing else fetched.  With 128 tokens to a wave the second
        batch of residual fragments has the place of the second fragment buffer, so that all of them are on their way at once."""
        seq, both = [], self.resid and self.TA == 4
        if self.resid:
            seq += self.residual_setup() + self.residual_loads(0, self.RES) + (self.residual_loads(1, self.FRAG[1]) if both else []) + self.identity()
        seq += [raw(f"s_waitcnt vmcnt({sum(x.kind == 'vmem' for x in seq)})", "wait"), raw("s_barrier", "barrier")]
        seq += self.frag_reads(0, 0, 0) + [raw("s_waitcnt lgkmcnt(0)", "wait")]
        if both:                                               # (the first step's last MFMAs have read their operands before the next fragments arrive)
            seq += self.pairs(0, True) + [nop(8)] + self.frag_reads(0, 0, 1) + [raw("s_waitcnt lgkmcnt(0)", "wait")] + self.pairs(0, False)
        else:
            seq += self.deal(self.pairs(0, True), self.frag_reads(1, 0, 1), []) + [raw("s_waitcnt lgkmcnt(0)", "wait")] + self.pairs(1, False)
        if self.resid:
            seq += [raw("s_waitcnt vmcnt(0)", "wait")] + self.residual_mfmas(0, self.RES) + (self.residual_mfmas(1, self.FRAG[1]) if both else [])
        return seq

    def body(self):
        pro = []
        e = pro.append
        for ks in range(2):
            for r, src, add in ((self.WADR + 2 * ks, "wfrag0", 0), (self.WADR + 2 * ks + 1, "wfrag0", 2 * self.WROWS * 128), (self.AADR + ks, "afrag0", 0)):
                e(valu(f"v_xor_b32 {V(r)}, {ks << 6}, %[{src}]", w=vr(r)))
                if add:
                    e(valu(f"v_add_u32 {V(r)}, {add}, {V(r)}", r=vr(r), w=vr(r)))
        # tile-load lane offsets: row 32 i + r0 of its matrix, clamped to the last valid row
        for i in range(self.NLD):
            is_w = i < self.NLW
            ofs = (self.WOFS + i) if is_w else (self.AOFS + i - self.NLW)
            row = (32 * i) % self.BN if is_w else 32 * (i - self.NLW)
            lim, stride = ("%[wlim]", "%[wstride]") if is_w else ("%[alim]", "%[astride]")
            e(valu(f"v_add_u32 {V(self.TMPV)}, {row}, %[r0]", w=vr(self.TMPV)))
            e(valu(f"v_min_i32 {V(self.TMPV)}, {lim}, {V(self.TMPV)}", r=vr(self.TMPV), w=vr(self.TMPV)))
            e(valu(f"v_mad_u32_u24 {V(ofs)}, {V(self.TMPV)}, {stride}, %[chunk]", r=vr(self.TMPV), w=vr(ofs)))
        ptrs = [(S_KPW, "w0base"), (S_KPA, "abase")] + ([(S_KPW2, "w1base")] if self.NW == 2 else [])
        for p, name in ptrs:
            e(salu(f"s_mov_b32 {S(p)}, %[{name}_lo]", w=sr(p)))
            e(salu(f"s_mov_b32 {S(p + 1)}, %[{name}_hi]", w=sr(p + 1)))
        e(salu(f"s_mov_b32 {S(S_CNT)}, %[kt]", w=sr(S_CNT)))
        e(salu(f"s_mov_b32 {S(S_LSTW)}, %[kt]", w=sr(S_LSTW)))
        e(salu(f"s_mov_b32 {S(S_LSTA)}, %[kt]", w=sr(S_LSTA)))
        pro += sum(self.loads(0, True) + self.loads(0, False), [])
        # a product of one k-tile leaves here: with the rings' other tiles on their way, which it does not read, it took 2 to 4 % longer
        pro += [salu("s_cmp_eq_u32 %[kt], 1", w=["scc"]), branch("s_cbranch_scc1 GSHORT_%=")]
        entry = list(pro)
        pro += sum(self.loads(1, True) + self.loads(1, False), [])
        n_res = 0
        if self.resid:
            pro += self.residual_setup() + self.residual_loads(0, self.RES) + self.identity()
            n_res = 4 * self.TW
        # only the first k-tile has to be there: the second one (and the residual fragments) may stay in flight until the first one's own wait
        e(raw(f"s_waitcnt vmcnt({self.NLD + n_res})", "wait"))
        e(raw("s_barrier", "barrier"))
        pro += self.frag_reads(0, 0, 0)
        dec = lambda: [salu(f"s_sub_u32 {S(S_CNT)}, {S(S_CNT)}, 1", r=sr(S_CNT), w=sr(S_CNT) + ["scc"]),
                       salu(f"s_cmp_eq_u32 {S(S_CNT)}, 0", r=sr(S_CNT), w=["scc"]), branch("s_cbranch_scc1 GDONE_%=")]
        seq, peeled = pro + self.k_tile(0, True), 1
        if self.resid:                                         # behind the first k-tile's wait, which covers their loads
            seq += self.residual_mfmas(0, self.RES)
        if self.resid and self.TA == 4:                        # (at least two k-tiles here)
            late = sum(1 for at, x in self.refill(0) if at >= 1 and x[0].kind == "vmem")
            seq += self.residual_loads(1, self.RES) + dec()[:1] + self.k_tile(1, False, late) + self.residual_mfmas(1, self.RES)
            peeled = 2
        seq = fix_hazards(seq) + dec() + [label("GLOOP_%=")]
        body = [self.k_tile(t, False) for t in range(peeled, peeled + self.period)]
        loop = sum((b + dec() for b in body), []) + [branch("s_branch GLOOP_%=")]
        seq += fix_hazards(loop, history=body[-2] + body[-1])
        seq += [label("GSHORT_%=")] + fix_hazards(self.only_k_tile(), history=entry)
        # drain the trailing loads; the accumulators are read by the compiler's code next: pad past the MFMA latency
        seq += [label("GDONE_%="), raw("s_waitcnt vmcnt(0) lgkmcnt(0)", "wait"), nop(8), nop(8)]
        n_mfma = 2 * sum(1 for x in body[0] if x.kind == "mfma")
        n_oth = sum(weight(x) for x in body[0] if x.kind not in ("mfma", "label"))
        print(f"wave tile {self.name}: k-tile of {n_mfma} MFMAs and {n_oth} other instructions, vgprs to v{self.LAST_V}", file=sys.stderr)
        return seq

    def function(self):
        n = self.NW * 2 * self.TW * self.NAF
        seq = self.body()
        out = [f"// wave tile of {2 * self.TW} x {2 * self.TA} MFMA tiles, {self.NW} weight matri{'x' if self.NW == 1 else 'ces'}"
               + ("; adds the residual tile to the accumulators" if self.resid else ""),
               f"__device__ __forceinline__ void gemm_mainloop_{self.name}(unsigned wfrag0, unsigned afrag0, unsigned r0, unsigned chunk,",
               "        int wlim, int alim, unsigned wstride, unsigned astride, unsigned kt, unsigned ldsw, uint64_t w0base,",
               f"        uint64_t w1base, uint64_t abase, f32x4 (&acc)[{self.NW}][{2 * self.TW}][{self.NAF}]"
               + (", unsigned rrow0, unsigned rcol0, unsigned rstride, const void* rbase" if self.resid else "") + ") {",
               "    f32x4 " + ", ".join(f"c{k}" for k in range(n)) + ";",
               "    const unsigned w0base_lo = (unsigned)w0base, w0base_hi = (unsigned)(w0base >> 32);",
               "    const unsigned w1base_lo = (unsigned)w1base, w1base_hi = (unsigned)(w1base >> 32);",
               "    const unsigned abase_lo = (unsigned)abase, abase_hi = (unsigned)(abase >> 32);",
               "    asm volatile("]
        out += ['        "' + x.text + '\\n"' for x in seq]
        # the last accumulators live in VGPRs: with all 256 accumulation registers taken by the outputs the compiler
        # spills some of them to scratch memory behind the loop (the residual form has no VGPRs to spare for that)
        in_vgprs = 0 if self.resid else N_ACC_IN_VGPRS
        out.append("        : " + ", ".join(f'[c{k}] "=&{"a" if k < n - in_vgprs else "v"}"(c{k})' for k in range(n)))
        ins = ['[wfrag0] "v"(wfrag0)', '[afrag0] "v"(afrag0)', '[r0] "v"(r0)', '[chunk] "v"(chunk)', '[wlim] "s"(wlim)',
               '[alim] "s"(alim)', '[wstride] "s"(wstride)', '[astride] "s"(astride)', '[kt] "s"(kt)', '[ldsw] "s"(ldsw)',
               '[w0base_lo] "s"(w0base_lo)', '[w0base_hi] "s"(w0base_hi)', '[abase_lo] "s"(abase_lo)', '[abase_hi] "s"(abase_hi)']
        if self.NW == 2:
            ins += ['[w1base_lo] "s"(w1base_lo)', '[w1base_hi] "s"(w1base_hi)']
        if self.resid:
            ins += ['[rrow0] "v"(rrow0)', '[rcol0] "v"(rcol0)', '[rstride] "s"(rstride)', '[rbase] "s"(rbase)']
        out.append("        : " + ", ".join(ins))
        clob = [f'"v{i}"' for i in range(self.LAST_V + 1)] + [f'"s{i}"' for i in range(FIRST_S, LAST_S + 1)] + ['"vcc"', '"scc"', '"memory"']
        out.append("        : " + ", ".join(clob) + ");")
        if self.NW == 1:
            out.append("    (void)w1base_lo; (void)w1base_hi;")
        k = 0
        for w in range(self.NW):
            for i in range(2 * self.TW):
                for j in range(self.NAF):
                    out.append(f"    acc[{w}][{i}][{j}] = c{k};")
                    k += 1
        out.append("}")
        return "\n".join(out) + "\n"


def main():
    here = sys.argv[1] if len(sys.argv) > 1 else os.path.dirname(os.path.abspath(__file__))   # output directory
    with open(os.path.join(here, "gemm_bf16_mainloops.inc"), "w") as f:
        f.write("// generated by gen_gemm_asm.py -- do not edit\n")
        for cfg in ((4, 4, 1), (2, 4, 2), (4, 2, 1), (2, 2, 2), (4, 4, 1, True), (4, 2, 1, True)):
            f.write("\n" + Shape(*cfg).function())


if __name__ == "__main__":
    main()
