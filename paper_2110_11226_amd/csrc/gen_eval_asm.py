"""Writes gp_eval_asm.h: the evaluation kernel's interpreter as gfx950 assembly,
one inline-assembly block per (rows per lane R, feature registers FREG), and the
adjoint's, one per R (AdjGen: the same instructions, those that record and apply
partial derivatives, and those that sum a constant's).

The block walks one compiled program (gp_eval_code.h) over one tile of 64 R
rows with threaded dispatch: every instruction word holds its handler's byte
offset from the handler table, each handler ends by jumping straight to the
next one, and the program's instructions sit in two vector registers (lane i
holds instruction i), so that fetching one is two v_readlane.  Stack slots,
features and the top of the stack have fixed registers, so an operation on
them is one vector instruction per row, with no copy and no indexed access.

What a compiler's switch costs here, per instruction: a compare tree (no jump
tables on this target), copies of each case's result into the loop's
registers, an indexed store of the top: 21 vector and 21 scalar instructions
and 9 branches for an addition on four rows.  Here: 4 vector instructions for
the rows, 2 for the fetch, 5 scalar.  Fitness of 256 programs of 1 to 200 nodes
on 16.8M rows: 104.4 ms with the switch, 75.6 ms here (28 features, log-loss,
500 programs, 1.1M rows: 18.6 and 10.0 ms).

The arithmetic bodies repeat, operation for operation, gp_crmath.h's sin, cos
and log and gp_device.hip's square root and division.  Inputs the common
paths do not cover, and the functions taken from the device library, leave
the block with a code (kExit...); the caller applies that operation to the
top and enters again.

Handler table order and register assignment are repeated in gp_eval_code.h
and gp_eval_asm.h by this generator.

Run from this directory: python gen_eval_asm.py
"""

SLOTS = 11          # stack entries below the top held in registers
STRIDE = 64         # bytes per handler
SRC_MAX = 9
FOPS = ["ADD", "SUB", "RSUB", "MUL", "DIV", "RDIV", "MAX", "MIN", "AT2", "RAT2"]
UNARY = ["NEG", "LOG", "SQRT", "SIN", "COS", "TAN", "ABS", "EXP", "INV", "SQ", "CUBE", "TANH", "ATAN", "CBRT"]
END, RELOAD, LOADY, SAVEL, LDT, LDB, UN = 0, 1, 2, 3, 4, 5, 6
SAVE = UN + len(UNARY)
LOADS = SAVE + SLOTS
SET = LOADS + SLOTS
# exit codes: 1 + unary index; these for the binary functions
EXIT_AT_TB, EXIT_AT_BT = 34, 35


def sections(freg):
    nsrc = 1 + max(1, freg)
    push = SET + nsrc
    fold = push + SLOTS * nsrc
    bin_ = fold + len(FOPS) * nsrc
    return dict(nsrc=nsrc, push=push, fold=fold, bin=bin_, count=bin_ + len(FOPS) * (SLOTS + 1))


class Gen:
    # scalar registers (see the operand list in emit_function)
    J, N0, N1, B, P, IDX, BLK, XC, T59, A, XB = 48, 50, 51, 52, 54, 55, 56, 58, 59, 60, 62
    INV, PA, PB, S5, C4, L2, L3, L5 = 64, 66, 68, 70, 72, 74, 76, 78
    LN2, C375, EPS, MASK, CLS, FOUR = 80, 82, 84, 85, 86, 87
    LD, Q0, Q1, Q2, LDS = 88, 90, 92, 94, 47

    def __init__(self, R, freg):
        self.R, self.freg = R, freg
        self.mem = freg == 0
        v = {1: 24, 2: 26, 4: 30}[R]

        def take(n):
            nonlocal v
            r = v
            v += n + (n & 1)
            return r
        self.base = v
        self.t = take(R)
        self.s = take(SLOTS * R)
        self.i = take(2)
        self.k = take(10)
        self.x = take(freg * R) if freg else None
        self.off = take(R) if self.mem else None
        self.p = take(R) if self.mem else None
        self.nb = min(R, 2)
        self.tmp = take(12 * self.nb)
        self.end = v
        self.RNDS, self.RNDC, self.S3, self.C2, self.L4 = (self.k + 2 * q for q in range(5))
        self.lines = []
        self.sec = sections(freg)

    # ---- emission helpers ----
    def o(self, s):
        self.lines.append(s)

    def label(self, n):
        self.o(f".L{n}_%=:")

    def br(self, n):
        self.o(f"s_branch .L{n}_%=")

    def hb(self):
        """Fetch the next instruction (its handler offset and payload)."""
        self.o(f"v_readlane_b32 s{self.N0}, v{self.i}, s{self.IDX}")
        self.o(f"v_readlane_b32 s{self.N1}, v{self.i + 1}, s{self.IDX}")
        self.o(f"s_add_u32 s{self.IDX}, s{self.IDX}, 1")

    def he(self):
        """Jump to it."""
        self.o(f"s_add_u32 s{self.J}, s{self.B}, s{self.N0}")
        self.o(f"s_addc_u32 s{self.J + 1}, s{self.B + 1}, 0")
        self.o(f"s_mov_b32 s{self.P}, s{self.N1}")
        self.o(f"s_setpc_b64 s[{self.J}:{self.J + 1}]")

    def rows(self, f):
        for j in range(self.R):
            self.o(f(j))

    def T(self, j):
        return f"v{self.t + j}"

    def S(self, k, j):
        return f"v{self.s + k * self.R + j}"

    def M(self, j):
        return f"v{self.tmp + j}"

    def src(self, q, j):
        if q == 0:
            return f"s{self.P}"
        return f"v{self.p + j}" if self.mem else f"v{self.x + (q - 1) * self.R + j}"

    # ---- handlers ----
    def handler(self, idx):
        self.o(f".p2align 6")
        self.label(f"h{idx}")

    def table(self):
        sec, R = self.sec, self.R
        wait = "s_waitcnt vmcnt(0)"
        h = 0

        def begin(want):
            nonlocal h
            assert h == want, (h, want)
            self.handler(h)
            h += 1
        begin(END)
        self.o(f"s_mov_b32 s{self.XC}, 0")
        self.br("exit")
        begin(RELOAD)
        self.br("reload")
        begin(LOADY)            # (the caller entered with it on top)
        self.hb()
        self.he()
        for want, name in ((SAVEL, "savel"), (LDT, "ldt"), (LDB, "ldb")):
            begin(want)
            self.hb()
            self.br(name)
        for u, name in enumerate(UNARY):
            begin(UN + u)
            self.hb()
            if name == "NEG":
                self.rows(lambda j: f"v_xor_b32 {self.T(j)}, 0x80000000, {self.T(j)}")
                self.he() if R < 4 else self.br("next")
            elif name == "ABS":
                self.rows(lambda j: f"v_and_b32 {self.T(j)}, 0x7fffffff, {self.T(j)}")
                self.he() if R < 4 else self.br("next")
            elif name == "SQ":
                self.rows(lambda j: f"v_mul_f32 {self.T(j)}, {self.T(j)}, {self.T(j)}")
                self.he()
            elif name == "CUBE":
                self.br("cube")
            elif name in ("LOG", "SQRT", "SIN", "COS", "INV"):
                self.br(name.lower())
            else:
                self.o(f"s_mov_b32 s{self.XC}, {1 + u}")
                self.br("leave")
        for k in range(SLOTS):
            begin(SAVE + k)
            self.hb()
            self.rows(lambda j: f"v_mov_b32 {self.S(k, j)}, {self.T(j)}")
            self.he()
        for k in range(SLOTS):
            begin(LOADS + k)
            self.hb()
            self.rows(lambda j: f"v_mov_b32 {self.T(j)}, {self.S(k, j)}")
            self.he()

        def from_src(q, op, tail="he"):
            """op on the rows with terminal q, then the next instruction (for a
            feature from memory, after requesting the next one)."""
            self.hb()
            if self.mem and q == 1:
                self.o(wait)
            self.rows(op)
            if self.mem and q == 1:
                self.br("m" + ("next" if tail == "he" else tail))
            elif tail == "he":
                self.he()
            else:
                self.br(tail)
        for q in range(sec["nsrc"]):
            begin(SET + q)
            from_src(q, lambda j: f"v_mov_b32 {self.T(j)}, {self.src(q, j)}")
        for k in range(SLOTS):
            for q in range(sec["nsrc"]):
                begin(sec["push"] + k * sec["nsrc"] + q)
                self.hb()
                if self.mem and q == 1:
                    self.o(wait)
                self.rows(lambda j: f"v_mov_b32 {self.S(k, j)}, {self.T(j)}")
                if R == 4:      # (the second half does not fit the handler)
                    self.br(f"set{q}")
                else:
                    self.rows(lambda j: f"v_mov_b32 {self.T(j)}, {self.src(q, j)}")
                    self.br("mnext") if self.mem and q == 1 else self.he()
        for f, name in enumerate(FOPS):
            for q in range(sec["nsrc"]):
                begin(sec["fold"] + f * sec["nsrc"] + q)
                simple = {"ADD": "v_add_f32", "SUB": "v_sub_f32", "RSUB": "v_subrev_f32", "MUL": "v_mul_f32"}
                if name in simple:
                    from_src(q, lambda j: f"{simple[name]} {self.T(j)}, {self.src(q, j)}, {self.T(j)}")
                else:
                    tail = {"DIV": "divmt", "RDIV": "divtm", "MAX": "max", "MIN": "min", "AT2": "atmt",
                            "RAT2": "attm"}[name]
                    from_src(q, lambda j: f"v_mov_b32 {self.M(j)}, {self.src(q, j)}", tail)
        for f, name in enumerate(FOPS):
            for k in range(SLOTS + 1):
                begin(sec["bin"] + f * (SLOTS + 1) + k)
                self.hb()
                b = (lambda j: self.S(k, j)) if k < SLOTS else self.M
                simple = {"ADD": ("v_add_f32", 0), "SUB": ("v_sub_f32", 0), "RSUB": ("v_sub_f32", 1),
                          "MUL": ("v_mul_f32", 0)}
                if name in simple:
                    op, rev = simple[name]
                    self.rows(lambda j: f"{op} {self.T(j)}, " + (f"{b(j)}, {self.T(j)}" if rev else f"{self.T(j)}, {b(j)}"))
                    self.he()
                else:
                    if k < SLOTS:
                        self.rows(lambda j: f"v_mov_b32 {self.M(j)}, {b(j)}")
                    self.br({"DIV": "divtm", "RDIV": "divmt", "MAX": "max", "MIN": "min", "AT2": "attm",
                             "RAT2": "atmt"}[name])
        assert h == sec["count"]

    # ---- out-of-line bodies ----
    def prefetch(self):
        """Requests the next feature from memory (payload: its index, negative: none)."""
        if not self.mem:
            return
        n = len(self.lines)
        self.o(f"s_cmp_lt_i32 s{self.P}, 0")
        self.o(f"s_cbranch_scc1 .Lnp{n}_%=")
        self.o(f"s_mul_i32 s{self.A}, s{self.P}, s{self.LD}")
        self.o(f"s_mul_hi_u32 s{self.A + 1}, s{self.P}, s{self.LD}")
        self.o(f"s_mul_i32 s{self.T59}, s{self.P}, s{self.LD + 1}")
        self.o(f"s_add_u32 s{self.A + 1}, s{self.A + 1}, s{self.T59}")
        self.o(f"s_add_u32 s{self.A}, s{self.A}, s{self.XB}")
        self.o(f"s_addc_u32 s{self.A + 1}, s{self.A + 1}, s{self.XB + 1}")
        self.rows(lambda j: f"global_load_dword v{self.p + j}, v{self.off + j}, s[{self.A}:{self.A + 1}]")
        self.label(f"np{n}")

    def lane(self, a):
        """This lane's index into v[a]."""
        self.o(f"v_mbcnt_lo_u32_b32 v{a}, -1, 0")
        self.o(f"v_mbcnt_hi_u32_b32 v{a}, -1, v{a}")

    def batches(self):
        return [list(range(a, min(a + self.nb, self.R))) for a in range(0, self.R, self.nb)]

    def interleave(self, per_row):
        """Rows' instruction lists merged round-robin."""
        for group in zip(*per_row):
            for x in group:
                if x:
                    self.o(x)

    def tp(self, b, q):
        """Temporary register q (0..11) of the batch's row b."""
        return self.tmp + 12 * b + q

    def pair(self, r):
        return f"v[{r}:{r + 1}]"

    def rare(self, name, code, cond):
        """Leaves for the caller's path if cond(j) holds on any row."""
        qs = [f"s[{self.Q0}:{self.Q0 + 1}]", f"s[{self.Q1}:{self.Q1 + 1}]", f"s[{self.Q2}:{self.Q2 + 1}]", "vcc"]
        for j in range(self.R):
            self.o(cond(j).format(q=qs[j]))
        for j in range(1, self.R):
            self.o(f"s_or_b64 {qs[0]}, {qs[0]}, {qs[j]}")
        if self.R == 1:
            self.o(f"s_cmp_lg_u64 {qs[0]}, 0")
        self.o(f"s_cbranch_scc1 .Lrare_{name}_%=")
        self.rare_exits.append((name, code))

    def sincos(self, name, rnd, deriv=None):
        """t = sin t or cos t; with `deriv`, its label, u = the derivative too."""
        self.label(deriv or name)
        self.o(f"s_mov_b32 s{self.T59}, 0x4b800000")
        u = UNARY.index(name.upper())
        self.rare(deriv or name, EXIT_ADJ_UN + u if deriv else 1 + u,
                  lambda j: f"v_cmp_ge_f32_e64 {{q}}, |{self.T(j)}|, s{self.T59}")
        for rows in self.batches():
            lists = []
            for b, j in enumerate(rows):
                P = lambda q: self.pair(self.tp(b, q))
                r = lambda q: f"v{self.tp(b, q)}"
                e = self.tp(b, 8)
                lists.append([
                    f"v_cvt_f64_f32 {P(0)}, {self.T(j)}",
                    f"v_fma_f64 {P(2)}, {P(0)}, s[{self.INV}:{self.INV + 1}], {self.pair(rnd)}",
                    f"v_lshlrev_b32_sdwa {r(6)}, s{self.FOUR}, {r(2)} dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0",
                    f"ds_read_b128 v[{e}:{e + 3}], {r(6)} offset:4096",
                    f"v_add_f64 {P(4)}, {P(2)}, -{self.pair(rnd)}",
                    f"v_fma_f64 {P(0)}, -{P(4)}, s[{self.PA}:{self.PA + 1}], {P(0)}",
                    f"v_fma_f64 {P(0)}, -{P(4)}, s[{self.PB}:{self.PB + 1}], {P(0)}",
                    f"v_mul_f64 {P(2)}, {P(0)}, {P(0)}",
                    f"v_fma_f64 {P(4)}, s[{self.S5}:{self.S5 + 1}], {P(2)}, {self.pair(self.S3)}",
                    f"v_fma_f64 {P(6)}, s[{self.C4}:{self.C4 + 1}], {P(2)}, {self.pair(self.C2)}",
                    f"v_fma_f64 {P(4)}, {P(2)}, {P(4)}, 1.0",
                    f"v_fma_f64 {P(6)}, {P(2)}, {P(6)}, 1.0",
                    f"v_mul_f64 {P(0)}, {P(0)}, {P(4)}",
                    f"s_waitcnt lgkmcnt({len(rows) - 1 - b})",
                    f"v_mul_f64 {P(4)}, {P(8)}, {P(6)}",
                    f"v_mul_f64 {P(6)}, {P(10)}, {P(6)}" if deriv else "",
                    f"v_fma_f64 {P(4)}, {P(10)}, {P(0)}, {P(4)}",
                    f"v_fma_f64 {P(6)}, -{P(8)}, {P(0)}, {P(6)}" if deriv else "",
                    f"v_cvt_f32_f64 {self.T(j)}, {P(4)}",
                    f"v_cvt_f32_f64 {self.U(j)}, {P(6)}" if deriv else ""])
            self.interleave(lists)
        self.he()

    def log(self):
        self.label("log")
        self.o(f"s_mov_b32 s{self.T59}, 0x7f800000")
        self.rare("log", 1 + UNARY.index("LOG"), lambda j: f"v_cmp_eq_f32_e64 {{q}}, |{self.T(j)}|, s{self.T59}")
        for rows in self.batches():
            lists = []
            for b, j in enumerate(rows):
                P = lambda q: self.pair(self.tp(b, q))
                r = lambda q: f"v{self.tp(b, q)}"
                e = self.tp(b, 8)
                q = (self.Q0, self.Q1)[b]
                lists.append([
                    f"v_lshrrev_b32 {r(2)}, 11, {self.T(j)}",
                    f"v_and_b32 {r(2)}, 0xff0, {r(2)}",
                    f"ds_read_b128 v[{e}:{e + 3}], {r(2)}",
                    f"v_cmp_gt_f32_e64 s[{q}:{q + 1}], |{self.T(j)}|, s{self.EPS}",
                    f"v_add_u32 {r(4)}, 0xffcb0000, {self.T(j)}",
                    f"v_bfi_b32 {r(0)}, s{self.MASK}, {self.T(j)}, 1.0",
                    f"v_frexp_exp_i32_f32 {r(4)}, {r(4)}",
                    f"v_cvt_f64_f32 {P(0)}, {r(0)}",
                    f"v_cvt_f64_i32 {P(4)}, {r(4)}",
                    f"s_waitcnt lgkmcnt({len(rows) - 1 - b})",
                    f"v_fma_f64 {P(0)}, {P(0)}, {P(8)}, -1.0",
                    f"v_fma_f64 {P(2)}, s[{self.L5}:{self.L5 + 1}], {P(0)}, {self.pair(self.L4)}",
                    f"v_mul_f64 {P(6)}, {P(0)}, {P(0)}",
                    f"v_fma_f64 {P(2)}, {P(2)}, {P(0)}, s[{self.L3}:{self.L3 + 1}]",
                    f"v_fma_f64 {P(4)}, {P(4)}, s[{self.LN2}:{self.LN2 + 1}], {P(10)}",
                    f"v_fma_f64 {P(2)}, {P(2)}, {P(0)}, s[{self.L2}:{self.L2 + 1}]",
                    f"v_fma_f64 {P(2)}, {P(6)}, {P(2)}, {P(0)}",
                    f"v_add_f64 {P(2)}, {P(4)}, {P(2)}",
                    f"v_cvt_f32_f64 {r(0)}, {P(2)}",
                    f"v_cndmask_b32_e64 {self.T(j)}, 0, {r(0)}, s[{q}:{q + 1}]"])
            self.interleave(lists)
        self.he()

    def sqrt(self):
        self.label("sqrt")
        for rows in self.batches():
            lists = []
            for b, j in enumerate(rows):
                P = lambda q: self.pair(self.tp(b, q))
                r = lambda q: f"v{self.tp(b, q)}"
                q = (self.Q0, self.Q1)[b]
                lists.append([
                    f"v_cvt_f64_f32_e64 {P(0)}, |{self.T(j)}|",
                    f"v_rsq_f64 {P(2)}, {P(0)}",
                    f"v_cmp_class_f64_e64 s[{q}:{q + 1}], {P(0)}, s{self.CLS}",
                    "s_nop 0" if b == 0 else "",
                    f"v_mul_f64 {P(4)}, {P(0)}, {P(2)}",
                    f"v_fma_f64 {P(2)}, -{P(4)}, {P(2)}, 1.0",
                    f"v_fma_f64 {P(6)}, {P(2)}, s[{self.C375}:{self.C375 + 1}], 0.5",
                    f"v_mul_f64 {P(2)}, {P(4)}, {P(2)}",
                    f"v_fma_f64 {P(4)}, {P(2)}, {P(6)}, {P(4)}",
                    f"v_cvt_f32_f64 {r(0)}, {P(4)}",
                    f"v_cndmask_b32_e64 {self.T(j)}, {r(0)}, |{self.T(j)}|, s[{q}:{q + 1}]"])
            self.interleave(lists)
        self.he()

    def minmax(self, name):
        """t = max(t, m) or min(t, m): a NaN operand is ignored, equal operands'
        sign bits are combined (-0 below +0)."""
        self.label(name)
        n = self.tmp + self.R
        qs = [f"s[{self.Q0}:{self.Q0 + 1}]", f"s[{self.Q1}:{self.Q1 + 1}]", f"s[{self.Q2}:{self.Q2 + 1}]", "vcc"]
        for j in range(self.R):
            self.o(f"v_cmp_eq_f32_e64 {qs[j]}, {self.T(j)}, {self.M(j)}")
        for j in range(self.R):
            t, m = self.T(j), self.M(j)
            # (operands quieted first: a signalling NaN would come through)
            self.o(f"v_max_f32 v{n}, {t}, {t}")
            self.o(f"v_max_f32 v{n + 1}, {m}, {m}")
            self.o(f"v_{name}_f32 v{n}, v{n}, v{n + 1}")
            self.o(f"v_{'and' if name == 'max' else 'or'}_b32 v{n + 1}, {t}, {m}")
            self.o(f"v_cndmask_b32_e64 {t}, v{n}, v{n + 1}, {qs[j]}")
        self.he()

    def div(self, name, num, den, other="1.0"):
        """t = |den| > eps ? num / den : other, the compiler's IEEE division."""
        self.label(name)
        for rows in self.batches():
            lists = []
            for b, j in enumerate(rows):
                d, r, n, q, e = (f"v{self.tmp + self.R + 5 * b + x}" for x in range(5))
                a, c = num(j), den(j)
                pq = (self.Q0, self.Q1)[b]
                vc = "vcc" if b == 0 else f"s[{self.Q2}:{self.Q2 + 1}]"
                lists.append([
                    f"v_cmp_gt_f32_e64 s[{pq}:{pq + 1}], |{c}|, s{self.EPS}",
                    f"v_div_scale_f32 {d}, s[{self.J}:{self.J + 1}], {c}, {c}, {a}",
                    f"v_div_scale_f32 {n}, {vc}, {a}, {c}, {a}",
                    f"v_rcp_f32 {r}, {d}",
                    "s_nop 0" if b == 0 else "",
                    f"v_fma_f32 {q}, -{d}, {r}, 1.0",
                    f"v_fma_f32 {r}, {q}, {r}, {r}",
                    f"v_mul_f32 {q}, {n}, {r}",
                    f"v_fma_f32 {e}, -{d}, {q}, {n}",
                    f"v_fma_f32 {q}, {e}, {r}, {q}",
                    f"v_fma_f32 {d}, -{d}, {q}, {n}"])
            self.interleave(lists)
            for b, j in enumerate(rows):
                d, r, n, q, e = (f"v{self.tmp + self.R + 5 * b + x}" for x in range(5))
                a, c = num(j), den(j)
                if b == 1:
                    self.o(f"s_mov_b64 vcc, s[{self.Q2}:{self.Q2 + 1}]")
                self.o(f"v_div_fmas_f32 {q}, {d}, {r}, {q}")
            for b, j in enumerate(rows):
                d, r, n, q, e = (f"v{self.tmp + self.R + 5 * b + x}" for x in range(5))
                self.o(f"v_div_fixup_f32 {q}, {q}, {den(j)}, {num(j)}")
            for b, j in enumerate(rows):
                q = f"v{self.tmp + self.R + 5 * b + 3}"
                pq = (self.Q0, self.Q1)[b]
                self.o(f"v_cndmask_b32_e64 {self.T(j)}, {other}, {q}, s[{pq}:{pq + 1}]")
        self.he()

    def bodies(self):
        R = self.R
        self.rare_exits = []
        self.label("next")
        self.he()
        if R == 4:
            for q in range(self.sec["nsrc"]):
                self.label(f"set{q}")
                self.rows(lambda j: f"v_mov_b32 {self.T(j)}, {self.src(q, j)}")
                self.br("mnext") if self.mem and q == 1 else self.he()
        if self.mem:
            self.label("mnext")
            self.prefetch()
            self.he()
        self.label("cube")
        self.rows(lambda j: f"v_mul_f32 {self.M(j)}, {self.T(j)}, {self.T(j)}")
        self.rows(lambda j: f"v_mul_f32 {self.T(j)}, {self.M(j)}, {self.T(j)}")
        self.he()
        a = self.tmp + 12 * self.nb - 1     # an address, clear of the operand in the first temporaries
        for name, ins in (("savel", "ds_write_b32 v{a}, {t} offset:{o}"), ("ldt", "ds_read_b32 {t}, v{a} offset:{o}"),
                          ("ldb", "ds_read_b32 {m}, v{a} offset:{o}")):
            self.label(name)
            self.lane(a)
            self.o(f"s_add_u32 s{self.T59}, s{self.P}, s{self.LDS}")
            self.o(f"v_lshl_add_u32 v{a}, v{a}, 2, s{self.T59}")
            self.rows(lambda j: ins.format(a=a, t=self.T(j), m=self.M(j), o=256 * j))
            if name != "savel":
                self.o("s_waitcnt lgkmcnt(0)")
            self.he()
        self.sincos("sin", self.RNDS)
        self.sincos("cos", self.RNDC)
        self.log()
        self.sqrt()
        for name, num, den in (("divtm", self.T, self.M), ("divmt", self.M, self.T)):
            if self.mem:
                self.label("m" + name)
                self.prefetch()
            self.div(name, num, den)
        self.div("inv", lambda j: "1.0", self.T, "0")
        for name in ("max", "min"):
            if self.mem:
                self.label("m" + name)
                self.prefetch()
            self.minmax(name)
        for name, code in (("attm", EXIT_AT_TB), ("atmt", EXIT_AT_BT)):
            if self.mem:
                self.label("m" + name)
                self.prefetch()
            self.label(name)
            self.o(f"s_mov_b32 s{self.XC}, {code}")
            self.br("leave")
        for name, code in self.rare_exits:
            self.label(f"rare_{name}")
            self.o(f"s_mov_b32 s{self.XC}, {code}")
            self.br("leave")
        self.label("reload")
        self.o(f"s_add_u32 s{self.BLK}, s{self.BLK}, 512")
        self.o(f"s_addc_u32 s{self.BLK + 1}, s{self.BLK + 1}, 0")
        self.lane(a)
        self.o(f"v_lshlrev_b32 v{a}, 3, v{a}")
        self.o(f"global_load_dwordx2 v[{self.i}:{self.i + 1}], v{a}, s[{self.BLK}:{self.BLK + 1}]")
        self.o(f"s_mov_b32 s{self.IDX}, 0")
        self.o("s_waitcnt vmcnt(0)")
        self.br("start")
        self.label("leave")
        # the instruction after this one was fetched: fetched again on entry
        self.o(f"s_sub_u32 s{self.IDX}, s{self.IDX}, 1")
        if self.mem:
            self.o("s_waitcnt vmcnt(0)")
        self.label("exit")

    def text(self):
        # everything the caller has in flight must have landed: the block counts
        # its own loads from zero
        self.o("s_waitcnt vmcnt(0) lgkmcnt(0)")
        self.o(f"s_getpc_b64 s[{self.B}:{self.B + 1}]")
        self.label("pc")
        self.o(f"s_add_u32 s{self.B}, s{self.B}, .Lh0_%=-.Lpc_%=")
        self.o(f"s_addc_u32 s{self.B + 1}, s{self.B + 1}, 0")
        self.label("start")
        self.hb()
        self.he()
        self.table()
        self.bodies()
        return self.lines


def pieces(n):
    """Register-tuple sizes covering n registers."""
    out = []
    for p in (32, 16, 8, 4, 2, 1):
        while n >= p:
            out.append(p)
            n -= p
    return out


def vec(n):
    return "float" if n == 1 else f"EvVec<float, {n}>"


def emit_function(R, freg):
    g = Gen(R, freg)
    lines = g.text()
    w = []
    # members: (name, type, first register, size, is_output)
    members = [("t", g.t, R)]
    at = g.s
    for q, n in enumerate(pieces(SLOTS * R)):
        members.append((f"s{q}", at, n))
        at += n
    outs = members + [("m", g.tmp, R)]
    ins = [("k0", g.k, 8), ("k1", g.k + 8, 2)]
    if freg:
        at = g.x
        for q, n in enumerate(pieces(freg * R)):
            ins.append((f"x{q}", at, n))
            at += n
    else:
        ins.append(("off", g.off, R))
        outs.append(("p", g.p, R))

    def vr(first, n):
        return f"{{v[{first}:{first + n - 1}]}}" if n > 1 else f"{{v{first}}}"
    w.append("template <>")
    w.append(f"struct Interp<{R}, {freg}> {{")
    w.append(f"    // v{g.base} .. v{g.end - 1}")
    for name, first, n in outs + ins:
        ty = "uint32_t" if name == "off" and n == 1 else \
            (f"EvVec<uint32_t, {n}>" if name == "off" else vec(n))
        w.append(f"    {ty} {name};")
    w.append("    EvVec<uint32_t, 2> ins;      // lane i: instruction i of the block")
    w.append("    uint32_t idx;                // next instruction of the block")
    w.append("    uint32_t blk0, blk1;         // address of the block")
    w.append("    uint32_t lds;                // LDS address of the wavefront's stack slots")
    w.append("    uint64_t xb, ld4;            // feature 0 of the tile's first row; bytes between features")
    w.append("    EvVec<uint32_t, 16> c0;      // scalar constants")
    w.append("    EvVec<uint32_t, 8> c1;")
    w.append("    __device__ __forceinline__ uint32_t run() {")
    w.append("        uint32_t code;")
    w.append("        asm volatile(")
    for ln in lines:
        w.append(f'            "{ln}\\n"')
    w.append("            : " + ", ".join(f'"+{vr(f, n)}"({nm})' for nm, f, n in outs) + ",")
    w.append(f'              "+{{v[{g.i}:{g.i + 1}]}}"(ins), "+{{s{g.IDX}}}"(idx), "+{{s{g.BLK}}}"(blk0), "+{{s{g.BLK + 1}}}"(blk1), "={{s{g.XC}}}"(code)')
    w.append("            : " + ", ".join(f'"{vr(f, n)}"({nm})' for nm, f, n in ins) + ",")
    w.append(f'              "{{s[64:79]}}"(c0), "{{s[80:87]}}"(c1), "{{s{g.LDS}}}"(lds)' +
             (f', "{{s[{g.XB}:{g.XB + 1}]}}"(xb), "{{s[{g.LD}:{g.LD + 1}]}}"(ld4)' if not freg else ""))
    clob = ["vcc", "scc", "memory"]
    clob += [f"s{q}" for q in (48, 49, 50, 51, 52, 53, 54, 59, 60, 61, 90, 91, 92, 93, 94, 95)]
    clob += [f"v{q}" for q in range(g.tmp + R, g.tmp + 12 * g.nb)]
    w.append("            : " + ", ".join(f'"{c}"' for c in clob) + ");")
    # (scalar registers all along; this tells the compiler that they are uniform)
    for nm in ("idx", "blk0", "blk1"):
        w.append(f"        {nm} = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>({nm})));")
    w.append("        return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(code)));")
    w.append("    }")
    w.append("};")
    return w


# ---------------------------------------------------------------------------
# The adjoint kernel's interpreter: the same table, then the instructions of
# reverse mode.  The forward part of a program records partial derivatives on
# a tape whose first TAPE entries are registers (written and read by handlers
# of their own: no address, no latency), the next TAPE_LDS lie in LDS and the
# rest in a per-wavefront memory area.  The reverse part carries the adjoint
# in the top's registers; slots hold the adjoints still to be carried back.
# ---------------------------------------------------------------------------
TAPE = 26
TAPE_LDS = 16
ACC = 8             # constants whose adjoints are summed in registers
ADJ_TAPE = ["PUTT", "PUTM", "PUTU", "GMUL", "MMUL"]
ADJ_ONE = ["SETMC", "SETMF", "MOVMT", "NEGMT", "MOVUT", "DINVM", "DINVT", "DNEGT", "DNEGM", "DSQRT", "SIND", "COSD", "CADDX"]
ADJ_UN = UNARY[UNARY.index("TAN"):]     # what the caller differentiates (the ones before have instructions of their own)
ADJ_BIN = ["MAXT", "MAXM", "MINT", "MINM", "ATTM", "ATMT"]
EXIT_ADJ_UN, EXIT_ADJ_BIN, EXIT_CADD = 64, 96, 112


def adj_sections():
    base = sections(0)["count"]
    sec = {}
    at = base
    for name, n in ([(t, TAPE) for t in ADJ_TAPE] + [(t + "L", 1) for t in ADJ_TAPE] + [(t + "G", 1) for t in ADJ_TAPE] +
                    [("LOADM", SLOTS), ("SAVEM", SLOTS)] + [(t, 1) for t in ADJ_ONE] + [("CADD", ACC)] +
                    [("UNX", len(ADJ_UN)), ("BINX", len(ADJ_BIN))]):
        sec[name] = at
        at += n
    sec["count"] = at
    return sec


class AdjGen(Gen):
    VM, GB = 36, 44     # row masks (R pairs); the wavefront's memory area

    def __init__(self, R):
        super().__init__(R, 0)
        v = self.end

        def take(n):
            nonlocal v
            r = v
            v += n + (n & 1)
            return r
        self.u = take(R)
        self.acc = take(2 * ACC)
        self.tape = take(TAPE * R)
        self.end = v
        self.adj = adj_sections()

    def U(self, j):
        return f"v{self.u + j}"

    def E(self, e, j):
        return f"v{self.tape + e * self.R + j}"

    def table(self):
        super().table()
        h = self.sec["count"]
        a = self.adj

        def begin(want):
            nonlocal h
            assert h == want, (h, want)
            self.handler(h)
            self.hb()
            h += 1
        on = {"PUTT": lambda j, e: f"v_mov_b32 {e}, {self.T(j)}", "PUTM": lambda j, e: f"v_mov_b32 {e}, {self.M(j)}",
              "PUTU": lambda j, e: f"v_mov_b32 {e}, {self.U(j)}",
              "GMUL": lambda j, e: f"v_mul_f32 {self.T(j)}, {self.T(j)}, {e}",
              "MMUL": lambda j, e: f"v_mul_f32 {self.M(j)}, {self.T(j)}, {e}"}
        for name in ADJ_TAPE:
            for e in range(TAPE):
                begin(a[name] + e)
                self.rows(lambda j: on[name](j, self.E(e, j)))
                self.he()
        for tier in "LG":
            for name in ADJ_TAPE:
                begin(a[name + tier])
                self.br(name.lower() + tier.lower())
        for k in range(SLOTS):
            begin(a["LOADM"] + k)
            self.rows(lambda j: f"v_mov_b32 {self.M(j)}, {self.S(k, j)}")
            self.he()
        for k in range(SLOTS):
            begin(a["SAVEM"] + k)
            self.rows(lambda j: f"v_mov_b32 {self.S(k, j)}, {self.M(j)}")
            self.he()
        for name in ADJ_ONE:
            begin(a[name])
            if name == "SETMC":
                self.rows(lambda j: f"v_mov_b32 {self.M(j)}, s{self.P}")
                self.he()
            elif name == "SETMF":
                self.o("s_waitcnt vmcnt(0)")
                self.rows(lambda j: f"v_mov_b32 {self.M(j)}, v{self.p + j}")
                self.br("mnext")
            elif name == "MOVMT":
                self.rows(lambda j: f"v_mov_b32 {self.M(j)}, {self.T(j)}")
                self.he()
            elif name == "MOVUT":
                self.rows(lambda j: f"v_mov_b32 {self.U(j)}, {self.T(j)}")
                self.he()
            elif name == "CADDX":
                self.o(f"s_mov_b32 s{self.XC}, {EXIT_CADD}")
                self.br("leave")
            else:
                self.br(name.lower())
        for k in range(ACC):
            begin(a["CADD"] + k)
            self.br(f"cadd{k}")
        for u, name in enumerate(ADJ_UN):
            begin(a["UNX"] + u)
            self.o(f"s_mov_b32 s{self.XC}, {EXIT_ADJ_UN + UNARY.index(name)}")
            self.br("leave")
        for q in range(len(ADJ_BIN)):
            begin(a["BINX"] + q)
            self.o(f"s_mov_b32 s{self.XC}, {EXIT_ADJ_BIN + q}")
            self.br("leave")
        assert h == a["count"]

    def recip(self, name, x):
        """u = |x| > eps ? 1 / x (hardware reciprocal) : 0."""
        self.label(name)
        n = self.tmp + self.R
        q = (self.Q0, self.Q1, self.Q2)
        for rows in [list(range(b, min(b + 3, self.R))) for b in range(0, self.R, 3)]:
            for i, j in enumerate(rows):
                self.o(f"v_cmp_gt_f32_e64 s[{q[i]}:{q[i] + 1}], |{x(j)}|, s{self.EPS}")
            for i, j in enumerate(rows):
                self.o(f"v_rcp_f32 v{n + i}, {x(j)}")
            self.o("s_nop 0")
            for i, j in enumerate(rows):
                self.o(f"v_cndmask_b32_e64 {self.U(j)}, 0, v{n + i}, s[{q[i]}:{q[i] + 1}]")
        self.he()

    def bodies(self):
        R, a = self.R, self.tmp + 12 * self.nb - 1
        n = self.tmp + R                    # temporaries beside the operand register
        leave = len(self.lines)
        super().bodies()
        # (the shared tail, from "reload" on, goes last)
        cut = next(i for i in range(leave, len(self.lines)) if self.lines[i].startswith(".Lreload_"))
        tail = self.lines[cut:]
        del self.lines[cut:]
        self.rare_exits = []
        self.label("negmt")
        self.rows(lambda j: f"v_xor_b32 {self.M(j)}, 0x80000000, {self.T(j)}")
        self.he()
        self.recip("dinvm", self.M)
        self.recip("dinvt", self.T)
        # u = u == 0 ? 0 : -x u u (a protected quotient has u = 0)
        for name, x in (("dnegt", self.T), ("dnegm", self.M)):
            self.label(name)
            for j in range(R):
                self.o(f"v_cmp_neq_f32_e64 vcc, 0, {self.U(j)}")
                self.o(f"v_mul_f32_e64 v{n}, -{x(j)}, {self.U(j)}")
                self.o(f"v_mul_f32 v{n}, v{n}, {self.U(j)}")
                self.o("s_nop 0")
                self.o(f"v_cndmask_b32_e32 {self.U(j)}, 0, v{n}, vcc")
            self.he()
        # u (the input x) and the top y = sqrt|x|: u = x == 0 ? 0 : copysign(1 / 2y, x)
        self.label("dsqrt")
        self.o(f"s_mov_b32 s{self.T59}, 0x7fffffff")
        for j in range(R):
            self.o(f"v_add_f32 v{n}, {self.T(j)}, {self.T(j)}")
            self.o(f"v_rcp_f32 v{n}, v{n}")
            self.o(f"v_cmp_neq_f32_e64 vcc, 0, {self.U(j)}")
            self.o(f"s_nop 0")
            self.o(f"v_bfi_b32 v{n}, s{self.T59}, v{n}, {self.U(j)}")
            self.o(f"v_cndmask_b32_e32 {self.U(j)}, 0, v{n}, vcc")
        self.he()
        self.sincos("sin", self.RNDS, "sind")
        self.sincos("cos", self.RNDC, "cosd")
        for k in range(ACC):
            self.label(f"cadd{k}")
            s0 = self.tmp + self.R + (self.R & 1)
            A = self.pair(self.acc + 2 * k)
            for j in range(R):
                self.o(f"v_cndmask_b32_e64 v{s0 + 4}, 0, {self.M(j)}, s[{self.VM + 2 * j}:{self.VM + 2 * j + 1}]")
                d = self.pair(s0 + (0 if j == 0 else 2))
                self.o(f"v_cvt_f64_f32 {d}, v{s0 + 4}")
                if j:
                    self.o(f"v_add_f64 {self.pair(s0)}, {self.pair(s0)}, {d}")
            self.o(f"v_add_f64 {A}, {A}, {self.pair(s0)}")
            self.he()
        regs = {"putt": self.T, "putm": self.M, "putu": self.U}
        for name in ADJ_TAPE:
            name = name.lower()
            self.label(name + "l")
            self.lane(a)
            self.o(f"s_add_u32 s{self.T59}, s{self.P}, s{self.LDS}")
            self.o(f"v_lshl_add_u32 v{a}, v{a}, 2, s{self.T59}")
            self.tape_op(name, regs, n, lambda j, r: f"ds_write_b32 v{a}, {r} offset:{256 * j}",
                         lambda j, r: f"ds_read_b32 {r}, v{a} offset:{256 * j}", "lgkmcnt(0)")
            self.label(name + "g")
            self.lane(a)
            self.o(f"v_lshlrev_b32 v{a}, 2, v{a}")
            self.o(f"s_add_u32 s{self.A}, s{self.GB}, s{self.P}")
            self.o(f"s_addc_u32 s{self.A + 1}, s{self.GB + 1}, 0")
            # (a read waits for the writes before it; a write's data stays put
            # until the wait at the next fetch, exit or read: the tape's
            # sources are only overwritten through the same registers in order)
            self.tape_op(name, regs, n,
                         lambda j, r: f"global_store_dword v{a}, {r}, s[{self.A}:{self.A + 1}] offset:{256 * j}",
                         lambda j, r: f"global_load_dword {r}, v{a}, s[{self.A}:{self.A + 1}] offset:{256 * j}",
                         "vmcnt(0)")
        for name, code in self.rare_exits:
            self.label(f"rare_{name}")
            self.o(f"s_mov_b32 s{self.XC}, {code}")
            self.br("leave")
        self.lines += tail

    def tape_op(self, name, regs, n, store, load, wait):
        if name in regs:
            self.rows(lambda j: store(j, regs[name](j)))
        else:
            if "vmcnt" in wait:
                self.o("s_waitcnt vmcnt(0)")
            self.rows(lambda j: load(j, f"v{n + j}"))
            self.o(f"s_waitcnt {wait}")
            self.rows(lambda j: f"v_mul_f32 {self.T(j) if name == 'gmul' else self.M(j)}, {self.T(j)}, v{n + j}")
        self.he()


def emit_adjoint(R):
    g = AdjGen(R)
    lines = g.text()
    w = []
    outs = []

    def group(name, first, n):
        at = first
        for q, m in enumerate(pieces(n)):
            outs.append((f"{name}{q}", at, m))
            at += m
    outs.append(("t", g.t, R))
    group("s", g.s, SLOTS * R)
    outs.append(("m", g.tmp, R))
    outs.append(("p", g.p, R))
    outs.append(("u", g.u, R))
    outs.append(("acc", g.acc, 2 * ACC))
    group("e", g.tape, TAPE * R)
    ins = [("k0", g.k, 8), ("k1", g.k + 8, 2), ("off", g.off, R)]

    def vr(first, n):
        return f"{{v[{first}:{first + n - 1}]}}" if n > 1 else f"{{v{first}}}"
    w.append("template <>")
    w.append(f"struct InterpAdjoint<{R}> {{")
    w.append(f"    // v{g.base} .. v{g.end - 1}")
    for name, first, n in outs + ins:
        ty = ("uint32_t" if n == 1 else f"EvVec<uint32_t, {n}>") if name == "off" else vec(n)
        w.append(f"    {ty} {name};")
    w.append("    EvVec<uint32_t, 2> ins;")
    w.append("    uint32_t idx, blk0, blk1, lds;")
    w.append("    uint32_t payload;            // of the instruction that left")
    w.append("    uint64_t xb, ld4, area;      // area: the wavefront's tape memory")
    w.append(f"    uint64_t mask[{R}];            // rows that count")
    w.append("    EvVec<uint32_t, 16> c0;")
    w.append("    EvVec<uint32_t, 8> c1;")
    w.append("    __device__ __forceinline__ uint32_t run() {")
    w.append("        uint32_t code;")
    w.append("        asm volatile(")
    for ln in lines:
        w.append(f'            "{ln}\\n"')
    w.append("            : " + ", ".join(f'"+{vr(f, n)}"({nm})' for nm, f, n in outs) + ",")
    w.append(f'              "+{{v[{g.i}:{g.i + 1}]}}"(ins), "+{{s{g.IDX}}}"(idx), "+{{s{g.BLK}}}"(blk0), "+{{s{g.BLK + 1}}}"(blk1), "={{s{g.XC}}}"(code), "={{s{g.P}}}"(payload)')
    w.append("            : " + ", ".join(f'"{vr(f, n)}"({nm})' for nm, f, n in ins) + ",")
    masks = ", ".join(f'"{{s[{g.VM + 2 * j}:{g.VM + 2 * j + 1}]}}"(mask[{j}])' for j in range(R))
    w.append(f'              "{{s[64:79]}}"(c0), "{{s[80:87]}}"(c1), "{{s{g.LDS}}}"(lds), "{{s[{g.XB}:{g.XB + 1}]}}"(xb), "{{s[{g.LD}:{g.LD + 1}]}}"(ld4), "{{s[{g.GB}:{g.GB + 1}]}}"(area), {masks}')
    clob = ["vcc", "scc", "memory"]
    clob += [f"s{q}" for q in (48, 49, 50, 51, 52, 53, 59, 60, 61, 90, 91, 92, 93, 94, 95)]
    clob += [f"v{q}" for q in range(g.tmp + R, g.tmp + 12 * g.nb)]
    w.append("            : " + ", ".join(f'"{c}"' for c in clob) + ");")
    for nm in ("idx", "blk0", "blk1", "payload"):
        w.append(f"        {nm} = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>({nm})));")
    w.append("        return static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(code)));")
    w.append("    }")
    w.append("};")
    return w


def main():
    out = ["// Generated by gen_eval_asm.py; do not edit.  The interpreter of the evaluation",
           "// kernel as gfx950 assembly (see the generator for its design).",
           "#pragma once", "", "#include <cstdint>", "",
           "template <typename T, int N>", "using EvVec = T __attribute__((ext_vector_type(N)));", "",
           "template <int R, int FREG>", "struct Interp;", ""]
    for R in (1, 2, 4):
        for freg in (0, 2, 8):
            out += emit_function(R, freg) + [""]
    out += ["// The adjoint kernel's: the same, then reverse mode.", "template <int R>", "struct InterpAdjoint;", ""]
    for R in (1, 2, 4):
        out += emit_adjoint(R) + [""]
    with open("gp_eval_asm.h", "w") as f:
        f.write("\n".join(out))
    code = ["// Generated by gen_eval_asm.py; do not edit.  The instruction stream that",
            "// the compile kernels write and the evaluation kernel's interpreter runs.",
            "//",
            "// An instruction is two words: the byte offset of its handler in the",
            "// interpreter's table, and a payload (a constant's bits; the index of the next",
            "// feature to fetch from memory, or -1; the byte offset of a stack slot in LDS).",
            "// Programs run in execution order; the value on top of the stack lives in its",
            "// own registers and entry e below it (from the bottom) in slot e.  The 64th",
            "// word pair of every 64 is kOpReload unless the program has ended.",
            "#pragma once", "", "#include <cstdint>", "",
            f"constexpr int kRegSlots = {SLOTS};        // slots held in registers; deeper ones live in LDS",
            f"constexpr uint32_t kOpBytes = {STRIDE};    // bytes per handler",
            "enum : uint32_t {",
            f"    kOpEnd = {END},", f"    kOpReload = {RELOAD},       // the next 64 instructions",
            f"    kOpLoadY = {LOADY},        // top = the row's target (first instruction only: the caller put it there)",
            f"    kOpSaveL = {SAVEL},        // LDS slot = top",
            f"    kOpLoadTopL = {LDT},     // top = LDS slot",
            f"    kOpLoadL = {LDB},        // operand register = LDS slot (for a kOpBin of slot kRegSlots)",
            f"    kOpUnary = {UN},        // + unary index: top = f(top)",
            f"    kOpSave = {SAVE},        // + slot: slot = top",
            f"    kOpLoadS = {LOADS},       // + slot: top = slot",
            f"    kOpSet = {SET},         // + source: top = source",
            "};",
            "// Sources: 0 a constant; 1 + f feature f in registers, or 1 the feature fetched",
            "// from memory (FREG = 0).  kPush + slot * n_src + source: slot = top, top = source.",
            "// kFold + op * n_src + source: top = source (op) top; kBin + op * (kRegSlots + 1) + slot:",
            "// top = top (op) slot; the reversed forms exchange the operands.",
            "struct EvalOps {", "    uint32_t n_src, push, fold, bin;", "};",
            "constexpr uint32_t eval_n_src(int freg) { return 1u + static_cast<uint32_t>(freg > 0 ? freg : 1); }",
            "constexpr EvalOps eval_ops(int freg) {",
            "    const uint32_t n = eval_n_src(freg), push = kOpSet + n, fold = push + kRegSlots * n;",
            f"    return EvalOps{{n, push, fold, fold + {len(FOPS)}u * n}};", "}",
            "enum : uint32_t {"]
    names = {"ADD": "Add", "SUB": "Sub", "RSUB": "SubRev", "MUL": "Mul", "DIV": "Div", "RDIV": "DivRev", "MAX": "Max",
             "MIN": "Min", "AT2": "Atan2", "RAT2": "Atan2Rev"}
    code += [f"    kB{names[n]} = {i}," for i, n in enumerate(FOPS)]
    code += ["};",
             "// What the interpreter leaves to its caller: 1 + unary index (top = f(top)), or one of",
             "// these on the top t and the operand register m.",
             "enum : uint32_t {", "    kExitEnd = 0,",
             f"    kExitAtan2TM = {EXIT_AT_TB},   // atan2(t, m)", f"    kExitAtan2MT = {EXIT_AT_BT},   // atan2(m, t)",
             "};", ""]
    names = {"PUTT": "PutT", "PUTM": "PutM", "PUTU": "PutU", "GMUL": "GMul", "MMUL": "MMul", "LOADM": "LoadM",
             "SAVEM": "SaveM", "SETMC": "SetMC", "SETMF": "SetMF", "MOVMT": "MovMT", "NEGMT": "NegMT", "MOVUT": "MovUT",
             "DINVM": "DInvM", "DINVT": "DInvT", "DNEGT": "DNegT", "DNEGM": "DNegM", "DSQRT": "DSqrt", "SIND": "SinD",
             "COSD": "CosD", "CADDX": "CAddX", "CADD": "CAdd", "UNX": "UnX", "BINX": "BinX"}
    code += ["// The adjoint kernel's instructions, after the table above (FREG = 0).  t is the",
             "// top (in the reverse part the adjoint), m the operand register, u a third.",
             "// kAPutT/M/U + entry: tape entry = t / m / u; kAGMul + entry: t *= entry; kAMMul +",
             "// entry: m = t * entry.  Entries from kTapeRegs on use the ...L forms (LDS, the",
             "// payload a byte offset), from kTapeRegs + kTapeLds on the ...G forms (memory).",
             "// kALoadM / kASaveM + slot: m = slot / slot = m.  kASetMC, kASetMF: m = constant, fetched",
             "// feature.  kAMovMT m = t, kANegMT m = -t, kAMovUT u = t.  kADInvM/T: u = protected",
             "// reciprocal of m / t; kADNegT/M: u = -t u u / -m u u; kADSqrt: u = d sqrt (u the input,",
             "// t the root); kASinD, kACosD: t = f(t), u = f'(t).  kACAdd + slot: the constant's adjoint",
             "// += m over the rows that count; kACAddX: the same by the caller (payload: slot).",
             "// kAUnX + unary index - that of tan: t = f(t), u = f'(t) by the caller; kABinX + kind: by the caller,",
             "// t = f of t and m, u = its derivative by t, m = by m (kinds: max and min with t, then",
             "// with m as the first operand, atan2(t, m), atan2(m, t)).",
             f"constexpr int kTapeRegs = {TAPE}, kTapeLds = {TAPE_LDS}, kAccRegs = {ACC};",
             f"constexpr uint32_t kAUnFirst = {UNARY.index('TAN')};", "enum : uint32_t {"]
    sec = adj_sections()
    for k, v in sec.items():
        if k == "count":
            continue
        base = k[:-1] if k[:-1] in ADJ_TAPE and k[-1] in "LG" else None
        code.append(f"    kA{names[base] + k[-1] if base else names[k]} = {v},")
    code += [f"    kAdjointOps = {sec['count']},", f"    kExitAdjUnary = {EXIT_ADJ_UN},", f"    kExitAdjBinary = {EXIT_ADJ_BIN},",
             f"    kExitCAdd = {EXIT_CADD},", "};", ""]
    with open("gp_eval_code.h", "w") as f:
        f.write("\n".join(code))


if __name__ == "__main__":
    main()
