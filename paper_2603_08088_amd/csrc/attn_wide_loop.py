"""Writes the tile loop of attn_wide_kernel (attention.hip) as one asm statement per variant: attn_wide_loop.h.

Why not HIP: the loop keeps 430 registers live in fixed places and interleaves three streams (matrix instructions, softmax,
LDS reads) at the grain of one instruction.  The compiler moves the scores through accumulation registers and issues the
fragment reads three or four products ahead of their use, whatever scheduling directives say.

One wavefront per SIMD, two 32-row chunks A and B.  A section is 64 matrix instructions of one chunk and, between them, the
softmax of the other:

    section A(t):  PV(A, t), QK(A, t + 1)   beside   softmax(B, t)        reads K(t + 1) from LDS for its own second half
    section B(t):  PV(B, t), QK(B, t + 1)   beside   softmax(A, t + 1)    reads V(t + 1) from LDS for section A(t + 1)

so a fragment is read once for 64 query rows, 32 ... 64 matrix instructions ahead of its first use.  The barrier that hands
over tiles stands at the head of section B(t): V(t + 1) and K(t + 2) have arrived, and every wavefront is done with V(t) and
K(t + 1), whose places are refilled with V(t + 4) and K(t + 5).

The first tiles of a split (up to three: the tree, a ragged end of the prefix) have masked keys: their scores' places in the
softmax go through the row's visibility bits.

The softmax takes no maximum: probabilities are 2^(score - reference), and their sum over the lane's keys, which is needed
anyway, tells whether the reference is too low (a sum above 2^8, or not a number).  Only then the row's maximum is taken, O
and l are rescaled and the probabilities computed again (`lift`).

The matrix instructions are 16x16x32: they move less accumulator data per product than 32x32x16, and the launch is limited by the
power.  64-lane layouts, l = lane % 16, g = lane / 16: A / B operand row | column l, contraction values 8 g ... 8 g + 7; accumulator
column l, rows 4 g + i.  A chunk's 32 query rows are two column blocks cb, so a lane has the rows l and 16 + l.

    S^T[key, q]: A = K[16 kb + l][32 ds + 8 g + j], B = Q[16 cb + l][the same]   score of key 16 kb + 4 g + i at S + 4 (2 kb + cb) + i
    O^T[d, q]:   contraction value j of g is key 32 ks + 4 g + j, and 12 more for j >= 4: B = the probabilities of the blocks kb = 2 ks
                 and 2 ks + 1 as they are, A = V^T by two transposing reads of four keys each; O + 4 (2 db + cb) + i, d = 16 db + 4 g + i

Registers: v0 ... v31 stay with the compiler.
"""
SA, SB = 32, 64            # scores
PA, PB = 96, 112           # probabilities, bf16 pairs: P + 4 (2 ks + cb) + 0 ... 3
VF = 128                   # V^T fragments: 16 x 4, 8 ks + db
TMP, PAIRS = 192, 6        # 6 pairs of temporaries
X = 204                    # 4 temporaries of lift and of the masked softmax
KADDR, VADDR = 208, 212    # LDS addresses of the fragments: by ds and by db % 4
KOFF, VOFF = 216, 220      # byte offsets of a lane's 16-byte pieces from the base of a 16-key block: 4 and 4
NM, L = 224, 228           # minus the references, sums of the probabilities: A's two column blocks, B's
SUM = 232                  # a tile's sums of the two column blocks; each is there four times
MASK = 240                 # visible keys, [tile][chunk]: bit 16 cb + 4 kb + i
ONES = 246                 # four bf16 ones
OA, OB, QA, QB, KF = 0, 64, 128, 160, 192    # accumulation registers: outputs, query fragments (2 ds + cb), K fragments (4 ds + kb)

# scalar registers of the loop
S_LEFT, S_STAGE, S_NEXT, S_DELTA, S_LIMIT, S_NINF = 40, 41, 42, 43, 44, 45
S_ID3, S_ID4, S_OFF, S_BASE, S_ID, S_LAST, S_BT, S_LIFT, S_TMP, S_IDX = 46, 47, 48, 50, 52, 53, 54, 56, 58, 59
S_KP, S_VP, S_STRIDE, S_LDS, S_SCALE, S_Q, S_MASKED, S_DONE, S_CHUNKS = 60, 62, 64, 65, 66, 67, 68, 69, 70
S_EMPTY = 72               # lanes whose rows have no finite score yet

TILE, STAGE, RING = 16384, 32768, 131072


class Out:
    def __init__(self):
        self.lines = []

    def __call__(self, *ops):
        for op in ops:
            self.lines.append(op)


def v(r, n=1):
    return f"v{r}" if n == 1 else f"v[{r}:{r + n - 1}]"


def a(r, n=1):
    return f"a{r}" if n == 1 else f"a[{r}:{r + n - 1}]"


def s(r, n=1):
    return f"s{r}" if n == 1 else f"s[{r}:{r + n - 1}]"


class Chunk:
    def __init__(self, name):
        first = name == "A"
        self.name = name
        self.S, self.P, self.O, self.Q = (SA, PA, OA, QA) if first else (SB, PB, OB, QB)
        self.nm, self.l, self.mask = (NM, L, MASK) if first else (NM + 2, L + 2, MASK + 1)


A, B = Chunk("A"), Chunk("B")
A2 = Chunk("A")            # chunk A with its probabilities where B's would be
A2.P = PB


# ---------------------------------------------------------------------------------------------------------------
# the three streams
# ---------------------------------------------------------------------------------------------------------------
def snake(outer):
    """The two column blocks for each of the outer blocks; neighbours share an operand."""
    return [(x, cb) for n, x in enumerate(outer) for cb in ((0, 1) if n % 2 == 0 else (1, 0))]


def qk_products(c):
    r = []
    for ds in range(4):
        for kb, cb in snake(range(4)):
            d = v(c.S + 4 * (2 * kb + cb), 4)
            r.append((f"v_mfma_f32_16x16x32_bf16 {d}, {a(KF + 4 * (4 * ds + kb), 4)}, {a(c.Q + 4 * (2 * ds + cb), 4)}, {'0' if ds == 0 else d}",
                      (("K", 4 * ds + kb), ("Q" + c.name, 2 * ds + cb))))
    return r


def pv_products(c):
    r = []
    for ks in range(2):
        for db, cb in snake(range(8)):
            o = a(c.O + 4 * (2 * db + cb), 4)
            r.append((f"v_mfma_f32_16x16x32_bf16 {o}, {v(VF + 4 * (8 * ks + db), 4)}, {v(c.P + 4 * (2 * ks + cb), 4)}, {o}", (("V", 8 * ks + db),)))
    return r


def k_reads():
    return [(f"ds_read_b128 {a(KF + 4 * (4 * ds + kb), 4)}, {v(KADDR + ds)} offset:{4096 * kb}", ("K", 4 * ds + kb))
            for ds in range(4) for kb in range(4)]


def q_reads(c, at):
    """From the addresses TMP ...; `at`: the chunk's place."""
    return [(f"ds_read_b128 {a(c.Q + 4 * (2 * ds + cb), 4)}, {v(TMP + ds)} offset:{at + 4096 * cb}", ("Q" + c.name, 2 * ds + cb))
            for ds in range(4) for cb in range(2)]


def v_reads():
    r = []
    for ks in range(2):
        for db in range(8):
            f = 8 * ks + db
            for half in range(2):
                r.append((f"ds_read_b64_tr_b16 {v(VF + 4 * f + 2 * half, 2)}, {v(VADDR + db % 4)} offset:{TILE + 8192 * ks + 4096 * half + 128 * (db // 4)}", ("V", f)))
    return r


def scores(c, i):
    """The registers and mask bits of the scores that become pair i of P."""
    ks, cb, r = i // 8, i // 4 % 2, i % 4
    kb, e = 2 * ks + r // 2, 2 * (r % 2)
    return c.S + 4 * (2 * kb + cb) + e, 16 * cb + 4 * kb + e, cb


def softmax(c, masked=False):
    """P = 2^(S * scale - reference) as bf16 pairs and the sum over them: a list of instructions, two or more apart where one
    needs the other (a transcendental result may be read by the second instruction behind it at the earliest, a matrix
    instruction may read what is two behind).

    The sum is over the rounded probabilities, the weights of the value product (over the unrounded ones the error against
    float64 grows by 0.5 %).  v_mfma_f32_4x4x4_16b_bf16 with ones adds up the four of two registers lane by lane; in groups of four,
    since a change between the two sizes of matrix instructions costs a dozen cycles.  Between 32x32x16 instructions a tile of the
    loop took 2574 cycles with it (one by one 2614), with v_dot2_f32_bf16 3046 (groups of 16: 2693), with the pairs taken apart for
    v_add_f32 2697."""
    fma, hide, exp, cvt, add = [], [], [], [], []
    for i in range(16):
        (s0, bit, cb), t0 = scores(c, i), TMP + 2 * (i % PAIRS)
        fma.append([f"v_fma_f32 {v(t0 + x)}, {v(s0 + x)}, {s(S_SCALE)}, {v(c.nm + cb)}" for x in range(2)])
        if masked:
            m0 = X + 2 * (i % 2)
            fma[-1] += [f"v_bfe_i32 {v(m0 + x)}, {v(c.mask)}, {bit + x}, 1" for x in range(2)]
            hide.append([f"v_bfi_b32 {v(t0 + x)}, {v(m0 + x)}, {v(t0 + x)}, {s(S_NINF)}" for x in range(2)])
        exp.append([f"v_exp_f32 {v(t0 + x)}, {v(t0 + x)}" for x in range(2)])
        cvt.append([f"v_cvt_pk_bf16_f32 {v(c.P + i)}, {v(t0)}, {v(t0 + 1)}"])
        add.append([])
        if i % 8 == 7:
            for half in range(2):
                for x in range(2):
                    total = v(SUM + 4 * x, 4)
                    add[-1].append(f"v_mfma_f32_4x4x4_16b_bf16 {total}, {v(ONES, 2)}, {v(c.P + i - 7 + 4 * x + 2 * half, 2)}, {total if i > 7 or half else 0}")
                if half == 0:
                    add[-1].append("s_nop 0")    # two wait states between those of a chain
    stages = (fma, hide, exp, cvt, add) if masked else (fma, exp, cvt, add)
    r = []
    for i in range(16 + len(stages) - 1):
        for lag, ops in enumerate(stages):
            if 0 <= i - lag < 16:
                r += ops[i - lag]
        if i == 16 + len(stages) - 2:
            r.insert(len(r) - 5, "s_nop 1")
    return r


def check(o, c, label, masked=False):
    """The tile's sums; out of line to `lift` where a reference is too low."""
    o("s_nop 4", f"v_add_f32 {v(X)}, {v(SUM)}, {v(SUM + 4)}", f"v_cmp_nle_f32 vcc, {v(X)}, {s(S_LIMIT)}",
      f"s_cbranch_vccnz .Llift_{label}%=", f".Llifted_{label}%=:", *[f"v_add_f32 {v(c.l + x)}, {v(c.l + x)}, {v(SUM + 4 * x)}" for x in range(2)])
    if masked:   # on to the next tile's bits; behind the masked tiles all keys are visible
        o(*[f"v_mov_b32 {v(c.mask + 2 * x)}, {v(c.mask + 2 * x + 2) if x < 2 else '-1'}" for x in range(3)])
    LIFTS.append((c, label, masked))


LIFTS = []


def lift(o, c, label, masked):
    """A row is in the lanes l, l + 16, l + 32, l + 48; one whose sum is above the limit in any of them moves its reference to the
    largest score of the tile.  The rows of its column block that do not are computed again to the same values; a column block
    without such a row is left alone.  Where that score is -inf too (products that overflow) the keys weigh nothing: the tile is
    computed against zero, and the reference stays where it was before the first finite score.

    The limit is the tile kernel's: it moves a reference that a score passes by 2^8, whose weight is then 1 and exact in bf16.  Every row that
    it would move moves here.  With a limit of 2^20 the error against float64 grew by up to 4 % (Q x 4; lse by 40 %).

    The matrix cores wait meanwhile.  B = 32, T = 128, P = 4096 in us, Q x 1, 3, 6, 12: tile kernel 295, 302, 308, 308; here 248, 269, 306,
    316; with both column blocks computed whichever row moved 246, 286, 329, 350."""
    # (O of a lone chunk is being written by the products just issued: more than 40 instructions pass before it is read here)
    o(f".Llift_{label}%=:")
    for cb in range(2):
        pairs = [i for i in range(16) if scores(c, i)[2] == cb]
        o(f"v_cmp_nle_f32 vcc, {v(SUM + 4 * cb)}, {s(S_LIMIT)}", f"s_cbranch_vccz .Lkeep_{label}{cb}%=",
          f"s_or_b32 {s(S_LIFT)}, vcc_lo, vcc_hi", f"s_lshr_b32 {s(S_TMP)}, {s(S_LIFT)}, 16",
          f"s_or_b32 {s(S_LIFT)}, {s(S_LIFT)}, {s(S_TMP)}", f"s_and_b32 {s(S_LIFT)}, {s(S_LIFT)}, 0xffff", f"s_lshl_b32 {s(S_TMP)}, {s(S_LIFT)}, 16",
          f"s_or_b32 {s(S_LIFT)}, {s(S_LIFT)}, {s(S_TMP)}", f"s_mov_b32 {s(S_LIFT + 1)}, {s(S_LIFT)}")
        for n, i in enumerate(pairs):
            at, bit, _ = scores(c, i)
            if masked:
                o(*[f"v_bfe_i32 {v(TMP + x)}, {v(c.mask)}, {bit + x}, 1" for x in range(2)])
                o(*[f"v_bfi_b32 {v(TMP + x)}, {v(TMP + x)}, {v(at + x)}, {s(S_NINF)}" for x in range(2)])
                at = TMP
            o(f"v_maximum3_f32 {v(X)}, {v(X if n else at)}, {v(at)}, {v(at + 1)}")
        for swap in ("32", "16"):
            o(f"v_mov_b32 {v(X + 1)}, {v(X)}", "s_nop 1", f"v_permlane{swap}_swap_b32 {v(X)}, {v(X + 1)}", "s_nop 1", f"v_max_f32 {v(X)}, {v(X)}, {v(X + 1)}")
        o(f"v_mul_f32 {v(X)}, {s(S_SCALE)}, {v(X)}",
          f"v_cndmask_b32_e64 {v(X)}, {v(c.nm + cb)}, -{v(X)}, {s(S_LIFT, 2)}",        # minus the new reference
          f"v_cmp_eq_f32_e64 {s(S_EMPTY, 2)}, {v(X)}, -{s(S_NINF)}", "s_nop 1",
          f"v_cndmask_b32_e64 {v(X)}, {v(X)}, 0, {s(S_EMPTY, 2)}",
          f"v_sub_f32 {v(X + 1)}, {v(X)}, {v(c.nm + cb)}", f"v_exp_f32 {v(X + 1)}, {v(X + 1)}", f"v_mov_b32 {v(c.nm + cb)}, {v(X)}",
          f"v_cmp_neq_f32 vcc, 0, {v(c.l + cb)}",
          f"v_cndmask_b32_e64 {v(X + 1)}, 1.0, {v(X + 1)}, {s(S_LIFT, 2)}", f"s_cbranch_vccz .Lempty_{label}{cb}%=",   # nothing to rescale yet
          f"v_mul_f32 {v(c.l + cb)}, {v(c.l + cb)}, {v(X + 1)}")
        for db in range(0, 8, 2):
            o_regs = [c.O + 4 * (2 * (db + x) + cb) + i for x in range(2) for i in range(4)]
            o(*[f"v_accvgpr_read_b32 {v(TMP + i)}, {a(r)}" for i, r in enumerate(o_regs)])
            o(*[f"v_mul_f32 {v(TMP + i)}, {v(TMP + i)}, {v(X + 1)}" for i in range(8)])
            o(*[f"v_accvgpr_write_b32 {a(r)}, {v(TMP + i)}" for i, r in enumerate(o_regs)])
        o(f".Lempty_{label}{cb}%=:")
        # `softmax` of the column block, four pairs of P at a time
        for ks in range(2):
            four = pairs[4 * ks:4 * ks + 4]
            total = v(SUM + 4 * cb, 4)
            o(*[f"v_fma_f32 {v(TMP + 2 * n + x)}, {v(scores(c, i)[0] + x)}, {s(S_SCALE)}, {v(c.nm + cb)}" for n, i in enumerate(four) for x in range(2)])
            if masked:
                for n, i in enumerate(four):
                    o(*[f"v_bfe_i32 {v(X + x)}, {v(c.mask)}, {scores(c, i)[1] + x}, 1" for x in range(2)])
                    o(*[f"v_bfi_b32 {v(TMP + 2 * n + x)}, {v(X + x)}, {v(TMP + 2 * n + x)}, {s(S_NINF)}" for x in range(2)])
            o(*[f"v_exp_f32 {v(TMP + n)}, {v(TMP + n)}" for n in range(8)])
            o(*[f"v_cvt_pk_bf16_f32 {v(c.P + i)}, {v(TMP + 2 * n)}, {v(TMP + 2 * n + 1)}" for n, i in enumerate(four)])
            for half in range(2):
                o("s_nop 2", f"v_mfma_f32_4x4x4_16b_bf16 {total}, {v(ONES, 2)}, {v(c.P + four[2 * half], 2)}, {total if ks or half else 0}")
        o(f"v_mov_b32 {v(X)}, 0x7f800000", f"v_cndmask_b32_e64 {v(c.nm + cb)}, {v(c.nm + cb)}, {v(X)}, {s(S_EMPTY, 2)}")
        o(f".Lkeep_{label}{cb}%=:")
    o("s_nop 4", f"s_branch .Llifted_{label}%=")


# ---------------------------------------------------------------------------------------------------------------
# tile loads: wavefront w brings the 16 keys 16 w ... of a tile, four loads of four rows for K and for V
# ---------------------------------------------------------------------------------------------------------------
def loads(what, place, nt):
    """Instructions, in order, for K or V of the tile at S_OFF; `place`: the ring place, a scalar register or a number."""
    base, voff, at = (S_KP, KOFF, 0) if what == "K" else (S_VP, VOFF, TILE)
    r = [f"s_add_u32 {s(S_BASE)}, {s(base)}, {s(S_OFF)}", f"s_addc_u32 {s(S_BASE + 1)}, {s(base + 1)}, {s(S_OFF + 1)}",
         f"s_add_u32 {s(S_TMP)}, {s(S_LDS)}, {place}"]
    for j in range(4):
        r.append(f"s_add_u32 m0, {s(S_TMP)}, {at + 1024 * j}")
        r.append("s_nop 0")
        r.append(f"global_load_lds_dwordx4 {v(voff + j)}, {s(S_BASE, 2)}{' nt' if nt else ''}")
    return r


def next_offset(paged, ident=S_ID):
    """S_OFF: byte offset of the wavefront's 16 keys of the next tile, from a block id (paged) or by counting on (contiguous)."""
    if paged:
        return [f"s_mul_i32 {s(S_OFF)}, {s(ident)}, {s(S_STRIDE)}", f"s_mul_hi_u32 {s(S_OFF + 1)}, {s(ident)}, {s(S_STRIDE)}"]
    return [f"s_add_u32 {s(S_OFF)}, {s(S_OFF)}, {s(S_STRIDE)}", f"s_addc_u32 {s(S_OFF + 1)}, {s(S_OFF + 1)}, 0"]


def fetch_id(dst, paged):
    """Block id of tile S_IDX, which then counts on; behind the last tile the last one's."""
    if not paged:
        return []
    return [f"s_min_u32 {s(S_TMP)}, {s(S_IDX)}, {s(S_LAST)}", f"s_lshl_b32 {s(S_TMP)}, {s(S_TMP)}, 4",
            f"s_load_dword {s(dst)}, {s(S_BT, 2)}, {s(S_TMP)}", f"s_add_u32 {s(S_IDX)}, {s(S_IDX)}, 1"]


# ---------------------------------------------------------------------------------------------------------------
# sections
# ---------------------------------------------------------------------------------------------------------------
class Reads:
    """LDS reads in flight, oldest first: how far the counter may stand when a fragment is needed."""

    def __init__(self):
        self.queue = []

    def issue(self, tag):
        self.queue.append(tag)

    def wait_for(self, o, tag):
        if tag not in self.queue:
            return
        last = len(self.queue) - 1 - self.queue[::-1].index(tag)
        newer = len(self.queue) - 1 - last
        o(f"s_waitcnt lgkmcnt({min(15, newer)})")
        del self.queue[:max(last + 1, len(self.queue) - 15)]


def slots(op):
    """Issue slots (4 cycles) of an instruction between matrix instructions."""
    return 2 if op.startswith("v_exp") else 0 if op.startswith("v_mfma") else int(op.split()[1]) + 1 if op.startswith("s_nop") else 1


def section(o, products, valu, reads, flying, extra=(), valu_from=2):
    """Matrix instructions with the other streams between them.  reads: (slot, instruction, tag); extra: (slot, instruction).

    A lone wavefront issues one instruction in four cycles, two of them in the shadow of a 16x16x32 product (64 products alone
    1048 cycles, with one or two v_fma_f32 behind each 1056 and 1061, with three 1317; two products and then four v_fma_f32: 1332; v_exp_f32
    counts twice).  There is more to issue than that, so what counts is that no product goes without its two: the vector stream
    follows the pace of all streams together, and fills up where the others leave a slot."""
    n = len(products)
    beside = [[] for _ in range(n)]
    for slot, ins, tag in reads:
        beside[slot].append((ins, tag))
    for slot, ins in extra:
        beside[slot].append((ins, None))
    total = sum(slots(ins) for ops in beside for ins, _ in ops) + sum(slots(op) for op in valu)
    pace, issued, done = max(2.0, total / n), 0, 0
    for i, (text, _) in enumerate(products):
        if i % 4 == 0:   # for four products at a time
            for _, need in products[i:i + 4]:
                for tag in need:
                    flying.wait_for(o, tag)
        o(text)
        here = 0
        for ins, tag in beside[i]:
            o(ins)
            here += slots(ins)
            if tag:
                flying.issue(tag)
        while i >= valu_from and done < len(valu) and (here < 2 or issued + here + slots(valu[done]) <= pace * (i + 1)):
            o(valu[done])
            here += slots(valu[done])
            done += 1
        issued += here
    o(*valu[done:])


def spread(ops, first, per_slot=1.0):
    return [(int(first + i / per_slot), op) for i, op in enumerate(ops)]


def section_a(o, flying, nm, masked=False):
    """PV(A, t), QK(A, t + 1) | softmax(B, t); K(t + 1) is read in the first half."""
    reads = [(2 * i, ins, tag) for i, (ins, tag) in enumerate(k_reads())]
    move = [f"v_add_u32 {v(VADDR + x)}, {s(S_DELTA)}, {v(VADDR + x)}" for x in range(4)]
    section(o, pv_products(A) + qk_products(A), softmax(B, masked), reads, flying, spread(move, 40, 0.5))
    check(o, B, f"B{nm}", masked)


def hand_over(o, nm, paged, nt, steady):
    """The head of section B(t): wait for V(t + 1) and K(t + 2), barrier, ask for V(t + 4) and K(t + 5).  steady: both of these
    exist; the scalar instructions that remain to be issued are returned."""
    if steady:
        o("s_waitcnt vmcnt(16) lgkmcnt(0)")
    else:   # towards the last tile: fewer loads are behind the ones that are needed
        o("s_waitcnt lgkmcnt(0)", f"s_cmp_gt_u32 {s(S_LEFT)}, 4", f"s_cbranch_scc1 .Lw16_{nm}%=", f"s_cmp_eq_u32 {s(S_LEFT)}, 4",
          f"s_cbranch_scc1 .Lw12_{nm}%=", f"s_cmp_eq_u32 {s(S_LEFT)}, 3", f"s_cbranch_scc1 .Lw4_{nm}%=", "s_waitcnt vmcnt(0)",
          f"s_branch .Lw_{nm}%=", f".Lw4_{nm}%=:", "s_waitcnt vmcnt(4)", f"s_branch .Lw_{nm}%=", f".Lw12_{nm}%=:", "s_waitcnt vmcnt(12)",
          f"s_branch .Lw_{nm}%=", f".Lw16_{nm}%=:", "s_waitcnt vmcnt(16)", f".Lw_{nm}%=:")
    o("s_barrier")
    ask_v, ask_k = loads("V", s(S_STAGE), nt), next_offset(paged) + loads("K", s(S_NEXT), nt) + fetch_id(S_ID, paged)
    scalar = []
    if steady:
        scalar += [op for op in ask_v + ask_k if op != "s_nop 0"]   # (a matrix instruction comes between)
    else:
        o(f"s_cmp_lt_u32 {s(S_LEFT)}, 5", f"s_cbranch_scc1 .Lnone_{nm}%=", *ask_v)
        o(f"s_cmp_lt_u32 {s(S_LEFT)}, 6", f"s_cbranch_scc1 .Lnone_{nm}%=", *ask_k)
        o(f".Lnone_{nm}%=:")
    # ring places of the next iteration
    return scalar + [f"s_mov_b32 {s(S_STAGE)}, {s(S_NEXT)}", f"s_add_u32 {s(S_NEXT)}, {s(S_NEXT)}, {STAGE}",
                     f"s_and_b32 {s(S_NEXT)}, {s(S_NEXT)}, {RING - 1}", f"s_sub_i32 {s(S_DELTA)}, {s(S_NEXT)}, {s(S_STAGE)}",
                     f"s_sub_u32 {s(S_LEFT)}, {s(S_LEFT)}, 1"]


def section_b(o, flying, nm, paged, nt, steady, masked=False):
    """PV(B, t), QK(B, t + 1) | softmax(A, t + 1); V(t + 1) is read as its fragments' last uses go by."""
    scalar = hand_over(o, nm, paged, nt, steady)
    flying.queue.clear()
    extra = spread(scalar, 0, 1.0)
    last = max([slot for slot, _ in extra])
    extra += spread([f"v_add_u32 {v(KADDR + x)}, {s(S_DELTA)}, {v(KADDR + x)}" for x in range(4)], max(last + 1, 40), 0.5)
    reads = [(2 * i + 1, ins, tag) for i, (ins, tag) in enumerate(v_reads())]
    section(o, pv_products(B) + qk_products(B), softmax(A, masked), reads, flying, extra)
    check(o, A, f"A{nm}", masked)


def after_v_reads():
    """The LDS reads in flight where section A(t) begins: those of V(t)."""
    flying = Reads()
    for _, tag in v_reads():
        flying.issue(tag)
    return flying


def more_tiles(o, nm, paged, nt):
    """Nobody reads Q or K(0) any more: places for K(3), V(3) and K(4)."""
    o("s_waitcnt lgkmcnt(0)", "s_barrier", f"s_cmp_lt_u32 {s(S_LEFT)}, 4", f"s_cbranch_scc1 .Lp2{nm}%=")
    o(*(next_offset(True, S_ID3) if paged else []), *loads("K", 3 * STAGE, nt), *loads("V", 3 * STAGE, nt))
    o(f"s_cmp_lt_u32 {s(S_LEFT)}, 5", f"s_cbranch_scc1 .Lp2{nm}%=", *next_offset(paged, S_ID4), *loads("K", s(S_STAGE), nt), f".Lp2{nm}%=:")


def second_tile(o, nm):
    """K(1) has arrived."""
    o(f"s_cmp_lt_u32 {s(S_LEFT)}, 5", f"s_cbranch_scc1 .Lp3{nm}%=", "s_waitcnt vmcnt(24)", f"s_branch .Lp4{nm}%=", f".Lp3{nm}%=:",
      "s_waitcnt vmcnt(0)", f".Lp4{nm}%=:", "s_barrier")


def first_reads():
    """Q of chunk A and K(0), by ds."""
    queries, keys = q_reads(A, 0), k_reads()
    return [r for ds in range(4) for r in queries[2 * ds:2 * ds + 2] + keys[4 * ds:4 * ds + 4]]


def one_chunk(o, paged, nt):
    """A wavefront with chunk A only: its softmax runs beside its own value product, the probabilities of every other tile in the place
    of chunk B's.

        QK(A, t + 1), V(t) read | barrier | PV(A, t) beside softmax(A, t + 1), K(t + 2) read

    Or with no chunk: it brings its share of the tiles."""
    fly = Reads()
    o(".Lnot_both%=:", f"s_cmp_eq_u32 {s(S_CHUNKS)}, 0", "s_cbranch_scc1 .Lno_chunk%=")
    o(*[f"v_add_u32 {v(TMP + ds)}, {s(S_Q)}, {v(KADDR + ds)}" for ds in range(4)])
    for ins, tag in first_reads():
        o(ins)
        fly.issue(tag)
    o(f"s_cmp_lg_u32 {s(S_DONE)}, 0", "s_cbranch_scc1 .Lnext_pass1%=", *[f"v_accvgpr_write_b32 {a(OA + i)}, 0" for i in range(64)], ".Lnext_pass1%=:")
    section(o, qk_products(A), [], [], fly)
    more_tiles(o, "o", paged, nt)
    o(*softmax(A, True))
    check(o, A, "Ao", True)
    o(f"s_cmp_lt_u32 {s(S_LEFT)}, 2", "s_cbranch_scc1 .Llast_A%=")
    second_tile(o, "o")
    o(*[f"v_add_u32 {v(KADDR + x)}, {s(S_DELTA)}, {v(KADDR + x)}" for x in range(4)], *[ins for ins, _ in k_reads()])

    def one_tile(now, then, nm, masked):
        flying = Reads()
        for _, tag in k_reads():
            flying.issue(tag)
        section(o, qk_products(then), [], [(i, ins, tag) for i, (ins, tag) in enumerate(v_reads())], flying)
        o(*[f"v_add_u32 {v(VADDR + x)}, {s(S_DELTA)}, {v(VADDR + x)}" for x in range(4)])
        o(*hand_over(o, nm, paged, nt, False))
        o(*[f"v_add_u32 {v(KADDR + x)}, {s(S_DELTA)}, {v(KADDR + x)}" for x in range(4)])
        # (behind the last tile the reads find an older one, and nothing uses them)
        section(o, pv_products(now), softmax(then, masked), [(2 * i, ins, tag) for i, (ins, tag) in enumerate(k_reads())], Reads())
        check(o, then, nm, masked)

    # the masked tiles, then the others, two tiles a turn
    for masked in (True, False):
        x = "m" if masked else "p"
        o(f".Lone_{x}%=:")
        for now, then, nm in ((A, A2, "A"), (A2, A, "B")):
            one_tile(now, then, f"1{nm}{x}", masked)
            o(f"s_cmp_lt_u32 {s(S_LEFT)}, 2", f"s_cbranch_scc1 .Llast_{'B' if nm == 'A' else 'A'}%=")
        if masked:
            o(f"s_sub_u32 {s(S_MASKED)}, {s(S_MASKED)}, 2", f"s_cmp_gt_i32 {s(S_MASKED)}, 0")
        o(f"s_cbranch_scc1 .Lone_m%=" if masked else "s_branch .Lone_p%=")
    for c, nm in ((A, "A"), (A2, "B")):
        o(f".Llast_{nm}%=:", *[ins for ins, _ in v_reads()])
        section(o, pv_products(c), [], [], after_v_reads())
        o("s_branch .Lend%=")

    o(".Lno_chunk%=:")
    more_tiles(o, "n", paged, nt)
    o(f"s_cmp_lt_u32 {s(S_LEFT)}, 2", "s_cbranch_scc1 .Lend%=")
    second_tile(o, "n")
    o(".Lnone%=:")
    o(*hand_over(o, "n", paged, nt, False))
    o(f"s_cmp_gt_u32 {s(S_LEFT)}, 1", "s_cbranch_scc1 .Lnone%=", "s_branch .Lend%=")


def program(paged, nt):
    """Tiles 0, 1, 2 are on their way to ring places 0, 1, 2 (of each all of K, then all of V), Q to place 3 and the 32 KiB behind it.  S_LEFT tiles in
    all, of which the first S_MASKED (at most 3) have masked keys.  S_CHUNKS: those of the wavefront that hold rows."""
    o = Out()
    LIFTS.clear()
    fly = Reads()
    o(f"s_mov_b32 {s(S_LIMIT)}, 0x43800000", f"s_mov_b32 {s(S_NINF)}, 0xff800000",       # 2^8, -inf
      f"v_mov_b32 {v(ONES)}, 0x3f803f80", f"v_mov_b32 {v(ONES + 1)}, 0x3f803f80",
      f"s_mov_b32 {s(S_STAGE)}, 0", f"s_mov_b32 {s(S_NEXT)}, {STAGE}", f"s_mov_b32 {s(S_DELTA)}, {STAGE}")
    if paged:
        o(f"s_cmp_lt_u32 {s(S_LEFT)}, 4", "s_cbranch_scc1 .Lfew%=", *fetch_id(S_ID3, True), *fetch_id(S_ID4, True), *fetch_id(S_ID, True), ".Lfew%=:")
    # Q and tile 0 have arrived
    o(f"s_cmp_lt_u32 {s(S_LEFT)}, 3", "s_cbranch_scc1 .Lp0%=", "s_waitcnt vmcnt(16)", "s_branch .Lp1%=", ".Lp0%=:", "s_waitcnt vmcnt(0)", ".Lp1%=:",
      "s_waitcnt lgkmcnt(0)", "s_barrier")
    o(f"s_cmp_lt_u32 {s(S_CHUNKS)}, 2", "s_cbranch_scc1 .Lnot_both%=")
    o(*[f"v_add_u32 {v(TMP + ds)}, {s(S_Q)}, {v(KADDR + ds)}" for ds in range(4)])
    for ins, tag in first_reads() + q_reads(B, 8192):
        o(ins)
        fly.issue(tag)
    zero = [f"v_accvgpr_write_b32 {a(OA + i)}, 0" for i in range(128)]
    flying, fly2 = Reads(), Reads()
    flying.queue, fly2.queue = list(fly.queue), list(fly.queue)
    o(f"s_cmp_lg_u32 {s(S_DONE)}, 0", "s_cbranch_scc1 .Lnext_pass%=")
    section(o, qk_products(A), zero, [], flying, valu_from=0)
    o("s_branch .Lp5%=", ".Lnext_pass%=:")
    section(o, qk_products(A), [], [], fly2)
    o(".Lp5%=:")
    fly.queue.clear()
    more_tiles(o, "", paged, nt)
    section(o, qk_products(B), softmax(A, True), [(i, ins, tag) for i, (ins, tag) in enumerate(v_reads())], fly)
    check(o, A, "Ap", True)
    o(f"s_cmp_lt_u32 {s(S_LEFT)}, 2", "s_cbranch_scc1 .Ltail%=")
    second_tile(o, "")
    o(*[f"v_add_u32 {v(KADDR + x)}, {s(S_DELTA)}, {v(KADDR + x)}" for x in range(4)])

    o(".Lmasked%=:", f"s_cmp_eq_u32 {s(S_MASKED)}, 0", "s_cbranch_scc1 .Lplain%=")
    flying = after_v_reads()
    section_a(o, flying, "e", True)
    section_b(o, flying, "e", paged, nt, False, True)
    o(f"s_sub_u32 {s(S_MASKED)}, {s(S_MASKED)}, 1", f"s_cmp_gt_u32 {s(S_LEFT)}, 1", "s_cbranch_scc1 .Lmasked%=", "s_branch .Ltail%=")

    o(".Lplain%=:", f"s_cmp_lt_u32 {s(S_LEFT)}, 6", "s_cbranch_scc1 .Ldrain%=")
    flying = after_v_reads()
    o(".p2align 6", ".Lloop%=:")
    section_a(o, flying, "m")
    section_b(o, flying, "m", paged, nt, True)
    o(f"s_cmp_gt_u32 {s(S_LEFT)}, 5", "s_cbranch_scc1 .Lloop%=")
    o(".Ldrain%=:")
    flying = after_v_reads()
    o(".Ldrain_loop%=:")
    section_a(o, flying, "d")
    section_b(o, flying, "d", paged, nt, False)
    o(f"s_cmp_gt_u32 {s(S_LEFT)}, 1", "s_cbranch_scc1 .Ldrain_loop%=")

    o(".Ltail%=:", f"s_cmp_gt_u32 {s(S_MASKED)}, 0", "s_cbranch_scc1 .Ltail_masked%=")
    for masked in (False, True):
        flying = after_v_reads()
        section(o, pv_products(A), softmax(B, masked), [], flying)
        check(o, B, f"Bt{int(masked)}", masked)
        section(o, pv_products(B), [], [], flying)
        o("s_branch .Lend%=", *([] if masked else [".Ltail_masked%=:"]))
    one_chunk(o, paged, nt)
    for c, label, masked in LIFTS:
        lift(o, c, label, masked)
    o(".Lend%=:", "s_waitcnt lgkmcnt(0)", "s_nop 15")   # no scalar load may arrive after the loop, in a register used otherwise
    return o.lines


def clobbers():
    owned = set(range(KADDR, L + 4))
    names = [f"v{r}" for r in [*range(32, SUM + 8), ONES, ONES + 1] if r not in owned]
    names += [f"a{r}" for r in range(QA, KF + 64)]
    names += [f"s{r}" for r in range(S_STAGE, S_KP) if r not in (S_OFF, S_OFF + 1, S_BT, S_BT + 1, S_IDX, S_LAST)]
    names += [f"s{r}" for r in range(S_EMPTY, S_EMPTY + 2)]
    return names + ["vcc", "scc", "memory"]   # m0: as everywhere, set before each use


def header():
    out = ["// Written by attn_wide_loop.py: the tile loop of attn_wide_kernel.  Not to be edited.", "#pragma once", ""]
    out.append("#define ETV_WIDE_CLOBBERS " + ", ".join(f'"{c}"' for c in clobbers()))
    for paged in (0, 1):
        for nt in (0, 1):
            out.append(f"#define ETV_WIDE_LOOP_{'PAGED' if paged else 'FLAT'}{'_NT' if nt else ''} \\")
            lines = program(bool(paged), bool(nt))
            out += [f'    "{l}\\n\\t" \\' for l in lines[:-1]] + [f'    "{lines[-1]}\\n"']
    return "\n".join(out) + "\n"

