"""The generated k-loops of the bf16 projections, run on the CPU: one lane's view of addresses, slots and fragments.  No GPU."""
import importlib.util
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_06447_amd", "csrc")


def load(name):
    spec = importlib.util.spec_from_file_location(name, os.path.join(CSRC, name + ".py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


class Wave:
    """Lane 0 of wave 0, all tile origins 0 (so a tile pointer is 128 times its k-tile).  What LDS and registers hold is tracked by name."""

    def __init__(self, shape, kt):
        self.sh, self.scc, self.now = shape, 0, 0
        self.s = {"%[kt]": kt, "%[ldsw]": 0}
        self.v, self.frag = {}, {}
        self.flying, self.landed, self.visible, self.lds, self.read_at = [], set(), set(), {}, {}
        self.pending, self.lgkm, self.safe = set(), -1, -1   # reads up to `safe`: waited for by every wave
        self.done = {}                                   # accumulator -> [(k-tile, k-step)]
        self.residual = {}                               # accumulator -> [(token tile, feature group, identity)]

    def value(self, x):
        if x in ("%[wfrag0]", "%[w0base_lo]", "%[w0base_hi]", "%[w1base_lo]", "%[w1base_hi]", "%[abase_lo]", "%[abase_hi]"):
            return 0
        if x == "%[afrag0]":
            return 3 * self.sh.WROWS * 128
        return self.s[x] if x in self.s else self.v[x] if x in self.v else int(x, 0)

    def step(self, text):
        op, args = (text.split(None, 1) + [""])[:2]
        a = [x.strip() for x in args.split(",")]
        self.now += 1
        if op == "s_mov_b32":
            self.s[a[0]] = self.value(a[1])
        elif op in ("s_add_u32", "s_sub_u32", "s_addc_u32"):
            r = self.value(a[1]) - self.value(a[2]) if op == "s_sub_u32" else self.value(a[1]) + self.value(a[2]) + (self.scc if op == "s_addc_u32" else 0)
            self.s[a[0]], self.scc = r & 0xffffffff, int(r < 0 or r > 0xffffffff)
        elif op == "s_cmp_gt_i32":
            x = self.value(a[0])
            self.scc = int((x - (1 << 32) if x >> 31 else x) > self.value(a[1]))
        elif op == "s_cmp_eq_u32":
            self.scc = int(self.value(a[0]) == self.value(a[1]))
        elif op == "s_cselect_b32":
            self.s[a[0]] = self.value(a[1]) if self.scc else self.value(a[2])
        elif op in ("v_xor_b32", "v_add_u32", "v_mov_b32"):
            if all(x in self.s or x in self.v or re.fullmatch(r"0x[0-9a-f]+|\d+|%\[[wa]frag0\]", x) for x in a[1:]):
                x = [self.value(y) for y in a[1:]]
                self.v[a[0]] = x[0] ^ x[1] if op == "v_xor_b32" else sum(x)
        elif op == "global_load_lds_dwordx4":
            ptr = int(re.match(r"s\[(\d+):", a[1]).group(1))
            assert self.s[f"s{ptr + 1}"] == 0 and self.s[f"s{ptr}"] % 128 == 0
            at, name = self.s["m0"], ({40: "w0", 42: "w1", 44: "a"}[ptr], self.s[f"s{ptr}"] // 128, int(a[0][1:]))
            assert at % 4096 == 0 and at < 163840
            # whatever was read from here was read by every wave: own reads waited for, then a barrier
            assert self.read_at.get(at, -1) <= self.safe, (text, at)
            self.lds[at] = name + (self.now,)
            self.flying.append(self.now)
        elif op == "global_load_dwordx4":
            off = int(a[2].split("offset:")[1]) if "offset:" in a[2] else 0
            base = int(re.match(r"v\[(\d+):", a[0]).group(1))
            self.frag[base] = ("r", int(a[1][1:]) - self.sh.ROFS, off // 64, self.now)
            self.flying.append(self.now)
        elif op == "ds_read_b128":
            adr, off = a[1].split(" offset:")
            at = self.v[adr] + int(off)
            ks, at = (at >> 6) & 1, at & ~127
            matrix, tile, ofs, when = self.lds[at // 4096 * 4096]
            assert when in self.visible, f"{text}: not there yet"
            row = at // 128 % 32 + 32 * (ofs - (self.sh.AOFS if matrix == "a" else self.sh.WOFS))
            base = int(re.match(r"v\[(\d+):", a[0]).group(1))
            self.frag[base] = (matrix, tile, ks, row)
            self.read_at[at // 4096 * 4096] = self.now
            self.pending.add(base)
        elif op == "s_waitcnt":
            m = re.search(r"vmcnt\((\d+)\)", text)
            if m:
                n = max(0, len(self.flying) - int(m.group(1)))
                self.landed |= set(self.flying[:n])
                self.flying = self.flying[n:]
            if "lgkmcnt(0)" in text:
                self.pending, self.lgkm = set(), self.now
        elif op == "s_barrier":
            self.safe, self.visible = self.lgkm, set(self.landed)
        elif op.startswith("v_mfma"):
            acc, x, y = a[0], int(a[1][2:].split(":")[0]), int(a[2][2:].split(":")[0])
            assert not {x, y} & self.pending, f"{text}: fragment not waited for"
            k = int(acc[3:-1])
            i, j = k // self.sh.NAF, k % self.sh.NAF
            if x >= self.sh.IDENT and self.sh.resid:
                _, tok, group, when = self.frag[y]
                assert when in self.landed and acc in self.done
                self.residual.setdefault(acc, []).append((tok, group, (x - self.sh.IDENT) // 4))
                return
            w, act = self.frag[x], self.frag[y]
            per = 2 * self.sh.TW
            # (in LDS the rows of a second weight matrix follow the first's; its wave-loads continue the numbering)
            assert w[0] == f"w{i // per}" and w[3] == i // per * self.sh.BN + i % per * 16, (text, w)
            assert act[0] == "a" and act[3] == 16 * j and act[1:3] == w[1:3], (text, w, act)
            assert (a[3] == "0") == (acc not in self.done)
            self.done.setdefault(acc, []).append(w[1:3])

    def run(self, seq):
        labels = {x.text[:-1]: n for n, x in enumerate(seq) if x.kind == "label"}
        pc = 0
        while pc < len(seq):
            x = seq[pc]
            pc += 1
            if x.kind == "branch":
                op, target = x.text.split()
                if op == "s_branch" or (op == "s_cbranch_scc1") == bool(self.scc):
                    pc = labels[target]
            elif x.kind not in ("label", "nop"):
                for text in x.text.split("\\n"):
                    self.step(text)


@pytest.mark.parametrize("cfg", [(4, 4, 1), (2, 4, 2), (4, 2, 1), (2, 2, 2), (4, 4, 1, True), (4, 2, 1, True)])
@pytest.mark.parametrize("kt", [1, 2, 3, 4, 5, 6, 7, 13])
def test_every_accumulator_sums_every_k_step(cfg, kt):
    """Each MFMA reads fragments of its own rows and of one k-step, from tiles that have landed in every wave's view; no slot is loaded into
    before all waves have read it; each accumulator takes all k-steps once, in order."""
    sh = load("gen_gemm_asm").Shape(*cfg)
    wave = Wave(sh, kt)
    wave.run(sh.body())
    assert len(wave.done) == sh.NW * 2 * sh.TW * sh.NAF and not wave.flying
    want = [(t, ks) for t in range(kt) for ks in range(2)]
    assert all(v == want for v in wave.done.values())
    if sh.resid:
        assert wave.residual == {f"%[c{i * sh.NAF + j}]": [(j, i // 2, i % 2)] for i in range(2 * sh.TW) for j in range(sh.NAF)}
