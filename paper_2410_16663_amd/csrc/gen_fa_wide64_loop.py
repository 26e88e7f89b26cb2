#!/usr/bin/env python3
"""Writes fa_attention_wide64_loop.inc: the check-free main loop of fa_fwd_wide64_kernel as one inline-assembly
block per storage type and number of row sums -- the software-pipelined form of the attention loop for waves of 64 query rows (four 16-row
blocks qb = 0 .. 3 that share every K and V fragment read from LDS).  One wave per SIMD, the whole register file.

Why assembly, and why generated: with one wave per SIMD nothing hides a wave's vector work but the wave itself, so
the instruction stream has to alternate -- one matrix instruction, then about as many vector / LDS / load
instructions as issue while it runs, then the next -- with three pieces of work in flight that do not depend on
each other.  The compiler's scheduler undoes such an interleaving and the rotating buffers confuse its register
allocator, hence fixed registers and a fixed order; the loop is regular, hence written by a script.  The build runs
this script (paper_2410_16663_amd/build.py); the .inc file is its output and is not kept under version control.

Register plan (per lane):
    a0   .. a127   O accumulators, O[qb][db] = a[32*qb + 4*db : +3]          (outputs of the block)
    a128 .. a191   Q fragments,    Q[qb][kb] = a[128 + 16*qb + 4*kb : +3]    (inputs)
    a192 .. a207   sums of the rounded exponentials, L[qb] = a[192 + 4*qb : +3], a row of the second product with ones
                   for V^T (all four registers the same; outputs)
    v0   .. v127   four unit buffers x four row blocks, X[b][qb] = v[32*b + 8*qb : +7]: unit u lives in X[u % 4], first
                   as logits (key block mb in registers 4*mb .. +3), then (overwritten in place) as packed exponentials
                   P = its first 4 registers
    v128 .. v143   four K fragments in flight;   v144 .. v159   four V^T fragments in flight
    v160+qb m_ref, v164+qb l_run (two sums: of the unrounded exponentials)    (outputs)
    v168 .. v171   the fragment of ones
    v172           K fragment address (input);   v173 .. v180   V^T fragment address per 16-row block of O^T (v173 input)
    v181, v182     per-lane byte offsets of the K and V loads from global memory (inputs)
    v183 .. v186   per row block of a unit: the sum of its exponentials (one sum: the largest)
    v187           causal limit of the lane's row in block 0, relative to the first key of its registers (input)
    v191, v192     temporaries;   v193 .. v200   per-lane offsets of the four loads per tensor
Scalar registers s60 .. s71 are scratch of the block.

A UNIT is 32 keys x the wave's 64 rows.  In step u the wave issues
    the 32 matrix instructions of unit u+1's logits   S(u+1) = K Q^T,
    the 32 matrix instructions of unit u-1's second product   O += V^T P(u-1), and 4 for its row of ones,
    and BETWEEN them the ~140 vector instructions of unit u's softmax   S(u) -> P(u)   (all row blocks), the
    LDS reads of the fragments three groups of four matrix instructions ahead, and this wave's share of a tile's loads.
The test "row sum <= 256" (which proves that no exponential exceeded 256, see the kernel) is computed at the end of the
step's vector work and branched on after its last matrix instruction; the rare other case runs a block out of line that
recomputes the unit's logits, takes the row maxima, moves the references, rescales the accumulators (through
v_accvgpr_read / write) and redoes the exponentials.

What issues when (measured, cycles, one wave per SIMD, all operands in registers): a 16 x 16 x 32 matrix instruction occupies
the matrix pipe for 16 and the vector port for 8 of them, so two vector instructions (4 each) or one v_exp_f32 (8) fit
behind it: 17.0 with two additions, 21.0 with three, 25.0 with four, 21.0 with v_fma and v_exp; a 32 x 32 x 16 (32) takes
six (33.0; eight: 41.0).  In the last 4 cycles of its port time something that is no vector instruction may issue (three
s_nop behind one: 17.0).  Four matrix instructions in a row, then eight additions: 89 instead of 68.  A dot product shares
the matrix pipe and stops it: 33.0 with one behind each matrix instruction, which is why no sum is taken with v_dot2c.
So each matrix instruction is followed by at most one LDS read or load instruction and by as many vector instructions as
are its even share of the step's, CAP cycles at least.

Units that reach past the causal limit of the wave's first row are masked before their vector work, in blocks out of line too
(two instructions per logit, 256 cycles): a wave walks its diagonal tile in the loop like the others.  (Its four waves' diagonal
tiles lie one tile apart; done by compiler-scheduled code each of them holds the other waves up at a barrier.)

LDS: four stages of (K tile, V tile); tile t lives in stage t % 4.  Barrier k (the k-th of the walk, the same count
as in the compiler-scheduled loop around this block) publishes tile k+1 and certifies that no wave reads tile k-1
any more; between barrier k and barrier k+1 every wave issues its share (four loads per tensor) of tile k+3.

Nothing issues in line that can issue behind a matrix instruction: the next unit's first key, whether it has to be masked and
whether it is the last are worked out there, and one branch a step, the one for the sums, stands for all three (counters and
branches between the steps cost 1%).

The reads ahead do not stop between steps: a step ends with reads of the next one's first fragments and begins with second
products, whose V^T fragments need no barrier, while the first K fragments of a tile just published are on their way.  The
barrier stands in an even step behind its last wait for V.  (Barrier and first K fragments between the steps, with the
logits first, left the matrix pipe idle for the LDS latency once a tile: 1 x 32 x 131072 103.4 ms, now 101.6; 8 x 32 x
8192 3776 us, 3742, fp16 3947, 3813; 512 queries on 32768 keys 250.5, 246.2.)

Steps: the block computes S(0), runs step 0 (no second product yet), then the steady loop -- eight steps per pass,
so that buffers and stages come round to where they started -- and leaves after step 2J-1 (J = number of tiles) through
one of four exits, each followed by the second product of the last unit.  Up to there it requests tiles up to J+2, or again
the last whole tile where there are no more, and reads K of tile J: what is not a tile of the walk goes to stages that nobody
reads and to fragments that nobody uses.

The reads ahead do not stop between steps: a step ends with reads of the next one's first fragments and begins with second
products, whose V^T fragments need no barrier, while the first K fragments of a tile just published are on their way.  The
barrier stands in an even step behind its last wait for V.  (Barrier and first K fragments between the steps, with the
logits first, left the matrix pipe idle for the LDS latency once a tile: 1 x 32 x 131072 103.4 ms, now 101.6; 8 x 32 x
8192 3776 us, 3742, fp16 3947, 3813; 512 queries on 32768 keys 250.5, 246.2.)

Steps: the block computes S(0), runs step 0 (no second product yet), then the steady loop -- eight steps per pass,
so that buffers and stages come round to where they started -- and leaves after step 2J-1 (J = number of tiles, even)
through one of two exits, each followed by the second product of the last unit.

Matrix instructions are 16 x 16 x 32: under the power limit the same flop cost less than as 32 x 32 x 16 (see mfma16 in
fa_device.inc), which pays for twice as many issue slots.  Four in a row share their K or V^T fragment, and neighbouring
groups run through the row blocks in opposite directions, so that consecutive ones mostly share an operand.

Hazards the hardware does not interlock, spaced by hand: 11 wait states between a matrix instruction and a vector
instruction touching its result (here: always a whole step apart, except in the blocks out of line, which wait);
results of v_exp_f32 are consumed several instructions later; 2 wait states around v_permlane32_swap.
"""
import os

KB, DB = 4, 8
KBLK = 1088
KTILEB = 16 * KBLK      # 17408
TILEB = 16384
NSTAGE = 4
QB, MB = 4, 2            # 16-row blocks of a wave, 16-key blocks of a unit
CAP = 8                 # cycles of vector instructions issued behind a matrix instruction (4: 1.00, 12: 0.98 of the speed)
NW = 4                  # waves per workgroup
NI = 16 // NW           # load instructions per wave, tensor and tile


def O(qb, db):
    r = 32 * qb + 4 * db
    return f"a[{r}:{r + 3}]"


def Q(qb, kb):
    r = 128 + 16 * qb + 4 * kb
    return f"a[{r}:{r + 3}]"


def LSUM(qb):
    return f"a[{192 + 4 * qb}:{192 + 4 * qb + 3}]"


def X(b, qb, mb):
    r = 32 * b + 8 * qb + 4 * mb
    return f"v[{r}:{r + 3}]"


def x(b, qb, i):
    return f"v{32 * b + 8 * qb + i}"


def P(b, qb):
    return X(b, qb, 0)


def KF(b):
    return f"v[{128 + 4 * b}:{128 + 4 * b + 3}]"


def VF(b):
    return f"v[{144 + 4 * b}:{144 + 4 * b + 3}]"


def VFlo(b):
    return f"v[{144 + 4 * b}:{144 + 4 * b + 1}]"


def VFhi(b):
    return f"v[{144 + 4 * b + 2}:{144 + 4 * b + 3}]"


M_REF = lambda qb: f"v{160 + qb}"
L_RUN = lambda qb: f"v{164 + qb}"
ONES = "v[168:171]"
KADDR = "v172"
VADDR = lambda db: f"v{173 + db}"
KVOFF, VVOFF = "v181", "v182"
SUM = lambda qb: f"v{183 + qb}"              # of a unit's exponentials (one sum: the largest)
LIMIT = "v187"
T4, T5 = "v191", "v192"
DMAOFF = lambda tensor, n: f"v{193 + 4 * tensor + n}"     # per-lane byte offset of load n of a K / V tile


class Gen:
    def __init__(self, bf16, two_sums):
        self.bf16 = bf16
        self.two_sums = two_sums
        self.mfma = "v_mfma_f32_16x16x32_bf16" if bf16 else "v_mfma_f32_16x16x32_f16"
        self.cvt = "v_cvt_pk_bf16_f32" if bf16 else "v_cvt_pk_f16_f32"
        self.out = []
        self.cold = []
        self.queue = []          # ids of LDS reads in flight, oldest first
        self.next_id = 0
        self.labels = {}
        self.nlabel = 0

    def emit(self, line):
        self.out.append(line)

    # ---- LDS reads and the waits for them (reads return in order)
    def lds_read(self, text, label):
        self.emit(text)
        self.queue.append(self.next_id)
        self.labels[self.next_id] = label
        self.next_id += 1
        return self.next_id - 1

    def wait_for(self, rid):
        if rid not in self.queue:
            return False
        i = self.queue.index(rid)
        n_after = len(self.queue) - 1 - i
        assert n_after <= 15
        self.emit(f"s_waitcnt lgkmcnt({n_after})")
        self.queue = self.queue[i + 1:]
        return True

    # fragment f of a unit's logits: key block f % MB, k-step f / MB
    def k_text(self, unit, f, slot):
        st, c = (unit >> 1) % NSTAGE, unit & 1
        off = st * KTILEB + (c * 8 + (f % MB) * 4) * KBLK + (f // MB) * 64
        return f"ds_read_b128 {KF(slot)}, {KADDR} offset:{off}"

    def k_read(self, unit, f):
        return self.lds_read(self.k_text(unit, f, f % 4), ("k", f))

    def v_read_lo(self, unit, db):
        st, c = (unit >> 1) % NSTAGE, unit & 1
        self.lds_read(f"ds_read_b64_tr_b16 {VFlo(db % 4)}, {VADDR(db)} offset:{st * TILEB + 8192 * c}", ("vlo", db))

    def v_read_hi(self, unit, db):
        st, c = (unit >> 1) % NSTAGE, unit & 1
        return self.lds_read(f"ds_read_b64_tr_b16 {VFhi(db % 4)}, {VADDR(db)} offset:{st * TILEB + 8192 * c + 4096}", ("vhi", db))

    def v_read(self, unit, db):
        self.v_read_lo(unit, db)
        return self.v_read_hi(unit, db)

    def qk(self, b, qb, f, slot):
        mb, kb = f % MB, f // MB
        return f"{self.mfma} {X(b, qb, mb)}, {KF(slot)}, {Q(qb, kb)}, {'0' if kb == 0 else X(b, qb, mb)}"

    def pv(self, b, qb, db):
        if db == "ones":
            return f"{self.mfma} {LSUM(qb)}, {ONES}, {P(b, qb)}, {LSUM(qb)}"
        return f"{self.mfma} {O(qb, db)}, {VF(db % 4)}, {P(b, qb)}, {O(qb, db)}"

    # ---- the vector work of one unit and row block, as a list of instructions (buffer b)
    def softmax_list(self, b, qb):
        """In place: logits X[b][qb] -> exponentials against the current reference, packed as P[b][qb]; leaves in SUM the sum
        of the exponentials (one sum: the largest).  The exponentials of the second group of four elements alternate with the
        additions / conversions of the first."""
        L = []
        acc = SUM(qb)

        def consume_parts(g):          # elements 4g .. 4g+3: two pairs -> [adds+cvt of pair 0], [.. pair 1]
            parts = []
            for pr in (2 * g, 2 * g + 1):          # pair pr = elements 2pr, 2pr+1 -> register pr
                a, bb = x(b, qb, 2 * pr), x(b, qb, 2 * pr + 1)
                one = []
                if self.two_sums:
                    if pr == 0:
                        one.append(f"v_add_f32 {acc}, {a}, {bb}")
                    else:
                        one.append(f"v_add_f32 {acc}, {acc}, {a}")
                        one.append(f"v_add_f32 {acc}, {acc}, {bb}")
                elif pr == 0:
                    one.append(f"v_max_f32 {acc}, {a}, {bb}")
                else:
                    one.append(f"v_max3_f32 {acc}, {acc}, {a}, {bb}")
                one.append(f"{self.cvt} {x(b, qb, pr)}, {a}, {bb}")
                parts.append(one)
            return parts

        for g in range(2):
            for i in range(4 * g, 4 * g + 4):
                L.append(f"v_fma_f32 {x(b, qb, i)}, {x(b, qb, i)}, %[c], -{M_REF(qb)}")
            ex = [f"v_exp_f32 {x(b, qb, i)}, {x(b, qb, i)}" for i in range(4 * g, 4 * g + 4)]
            if g == 0:
                L += ex
            else:
                p0, p1 = consume_parts(0)
                L += [ex[0]] + p0 + [ex[1]] + p1 + [ex[2], ex[3]]
        p0, p1 = consume_parts(1)
        return L + p0 + p1

    def softmax_all(self, b):
        """The four row blocks' lists, interleaved an instruction at a time (they share no register)."""
        S = [self.softmax_list(b, qb) for qb in range(QB)]
        L = []
        for i in range(len(S[0])):
            for q in range(QB):
                L.append(S[q][i])
        return L

    def pending_sums(self):
        """Adds the previous unit's sums (left in the temporaries by its vector work) to the running sums: the first
        vector instructions of the next step, or of the drain."""
        return [f"v_add_f32 {L_RUN(qb)}, {L_RUN(qb)}, {SUM(qb)}" for qb in range(QB)] if self.two_sums else []

    def check_list(self):
        """The test "the sum over all row blocks <= 256" (one sum: the largest), which proves that no exponential exceeded 256,
        leaving the outcome in vcc: the last vector instructions of a step."""
        if self.two_sums:
            L = [f"v_add_f32 {T4}, {SUM(0)}, {SUM(1)}", f"v_add_f32 {T5}, {SUM(2)}, {SUM(3)}", f"v_add_f32 {T4}, {T4}, {T5}"]
        else:
            L = [f"v_max_f32 {T4}, {SUM(0)}, {SUM(1)}", f"v_max3_f32 {T4}, {T4}, {SUM(2)}, {SUM(3)}"]
        L.append(f"v_cmp_nge_f32 vcc, 0x43800000, {T4}")             # not (256 >= sum): also true for inf and NaN
        return L

    def mask_lines(self, b, first_key):
        """Hides the logits of X[b] past each row's causal limit; first_key: the scalar register with the unit's first key.
        Register mb, r of row block qb is key 16 mb + r of those the limit counts from."""
        L = [f"v_subrev_u32 {T4}, {first_key}, {LIMIT}", f"v_mov_b32 {T5}, 0xff800000"]
        for qb in range(QB):
            for i in range(4 * MB):
                L += [f"v_cmp_gt_i32 vcc, {16 * (i // 4) + i % 4 - 16 * qb}, {T4}",
                      f"v_cndmask_b32 {x(b, qb, i)}, {x(b, qb, i)}, {T5}, vcc"]
        return L

    def finish_sums(self, unit):
        """After the step's last matrix instruction: if the sum exceeded 256, a block out of line computes the row blocks'
        logits again, moves the references up to the row maxima, rescales, and redoes the exponentials.  The same branch is
        taken (s[64:65]) where the next unit has to be masked, which happens there too, and where there is none."""
        e = self.emit
        b = unit % 4
        k = self.nlabel
        self.nlabel += 1
        e(f"s_cbranch_vccnz .Lfw64_redo_{k}_%=")
        e(f".Lfw64_back_{k}_%=:")
        # ---- the block out of line
        main, self.out = self.out, []
        e(f".Lfw64_redo_{k}_%=:")
        e(self.check_list()[-1])
        e("s_and_b64 vcc, vcc, exec")
        e("s_nop 3")
        e(f"s_cbranch_vccz .Lfw64_next_{k}_%=")
        e("s_waitcnt lgkmcnt(0)")
        for f in range(MB * KB):
            e(self.k_text(unit, f, 3))               # (slot 3 is free between steps)
            e("s_waitcnt lgkmcnt(0)")
            for qb in range(QB):
                e(self.qk(b, qb, f, 3))
            e("s_nop 7")
        e("s_nop 15")
        e("s_nop 3")
        e("s_sub_u32 s68, s66, 32")
        e("s_cmp_lt_i32 s68, s70")
        e(f"s_cbranch_scc1 .Lfw64_free_{k}_%=")
        for ln in self.mask_lines(b, "s68"):
            e(ln)
        e(f".Lfw64_free_{k}_%=:")
        if unit == 0:
            # the walk's first reference is the maximum over the whole first tile, as in the other kernels: the key that sets it
            # has a probability of 1, without rounding (over 32 keys the results are 0.1 to 0.2% further from 64 bits)
            e("s_cmp_lt_i32 s66, s70")
            e(f"s_cbranch_scc1 .Lfw64_tile_{k}_%=")
            for ln in self.mask_lines(1, "s66"):
                e(ln)
            e(f".Lfw64_tile_{k}_%=:")
        for qb in range(QB):
            X8 = [x(b, qb, i) for i in range(8)] + ([x(1, qb, i) for i in range(8)] if unit == 0 else [])
            e(f"v_max3_f32 {T4}, {X8[0]}, {X8[1]}, {X8[2]}")
            for i in range(3, len(X8) - 1, 2):
                e(f"v_max3_f32 {T4}, {T4}, {X8[i]}, {X8[i + 1]}")
            e(f"v_max_f32 {T4}, {T4}, {X8[-1]}")
            for swap in ("v_permlane32_swap_b32_e32", "v_permlane16_swap_b32_e32"):   # the lane groups hold different keys of one query
                e(f"v_mov_b32 {T5}, {T4}")
                e("s_nop 1")
                e(f"{swap} {T4}, {T5}")
                e("s_nop 1")
                e(f"v_max_f32 {T4}, {T4}, {T5}")
            e(f"v_mul_f32 {T4}, %[c], {T4}")                # in log2 units
            e(f"v_cmp_gt_f32 vcc, {T4}, {M_REF(qb)}")
            e(f"v_sub_f32 {T5}, {M_REF(qb)}, {T4}")
            e(f"v_exp_f32 {T5}, {T5}")
            e(f"v_cndmask_b32 {M_REF(qb)}, {M_REF(qb)}, {T4}, vcc")
            e("s_nop 1")
            e(f"v_cndmask_b32 {T5}, 1.0, {T5}, vcc")
            if self.two_sums:
                e(f"v_mul_f32 {L_RUN(qb)}, {T5}, {L_RUN(qb)}")
            # the accumulators live in AGPRs: out, times alpha, back in -- four at a time through the K fragment
            # registers of slot 3 (free here); the second products issued earlier in this step have long retired
            # (the 20 wait states above), and the matrix instructions that follow read them as their C operand
            tmp = [f"v{128 + 12 + i}" for i in range(4)]
            for r0 in [4 * DB * qb + 4 * db for db in range(DB)] + [192 + 4 * qb]:
                for i in range(4):
                    e(f"v_accvgpr_read_b32 {tmp[i]}, a{r0 + i}")
                e("s_nop 0")
                for i in range(4):
                    e(f"v_mul_f32 {tmp[i]}, {T5}, {tmp[i]}")
                e("s_nop 0")
                for i in range(4):
                    e(f"v_accvgpr_write_b32 a{r0 + i}, {tmp[i]}")
            for ln in self.softmax_list(b, qb):
                e(ln)
                e("s_nop 0")       # (a result of v_exp is read two or more instructions later)
        # (the fragments read ahead have landed: the main path's waits find fewer reads in flight)
        e(f".Lfw64_next_{k}_%=:")
        if unit & 1:
            e("s_cmp_ge_i32 s66, s67")
            e(f"s_cbranch_scc1 .Lfw64_drain_{unit % 8}_%=")
        e("s_nop 15")
        e("s_cmp_lt_i32 s66, s70")
        e(f"s_cbranch_scc1 .Lfw64_back_{k}_%=")
        for ln in self.mask_lines((unit + 1) % 4, "s66"):
            e(ln)
        e(f"s_branch .Lfw64_back_{k}_%=")
        self.cold += self.out
        self.out = main

    def dma_list(self, tile):
        """This wave's share of the loads of a tile, then the advance of the two tile pointers s[60:61] / s[62:63] as long
        as there are whole tiles (s69: how many), to be spread over a step.  (Between m0's new value and the load that reads it something else has to issue.)"""
        st = tile % NSTAGE
        G = []
        for tensor in (0, 1):
            ptr = "s[60:61]" if tensor == 0 else "s[62:63]"
            for n in range(NI):
                if tensor == 0:
                    G.append(f"s_add_u32 m0, %[ldsk], {st * KTILEB + NW * n * KBLK}")
                else:
                    G.append(f"s_add_u32 m0, %[ldsv], {st * TILEB + NW * n * 1024}")
                G.append(f"global_load_lds_dwordx4 {DMAOFF(tensor, n)}, {ptr} offset:0")
        G += ["s_sub_u32 s69, s69, 1", "s_cmp_ge_i32 s69, 0", f"s_cselect_b32 s68, {TILEB}, 0"]
        G += ["s_add_u32 s60, s60, s68", "s_addc_u32 s61, s61, 0", "s_add_u32 s62, s62, s68", "s_addc_u32 s63, s63, 0"]
        return G

    @staticmethod
    def check_distances(lines):
        """In a stream of vector instructions (whatever is issued in between only widens the distances) a result of v_exp is
        read two or more instructions later, which the hardware does not watch."""
        exp_at = {}
        for pos, ln in enumerate(lines):
            op, _, rest = ln.partition(" ")
            regs = [r.strip().lstrip("-") for r in rest.split(",")]
            for r in regs[1:]:
                assert pos - exp_at.get(r, -2) >= 2, ln
            exp_at.pop(regs[0], None)
            if op == "v_exp_f32":
                exp_at[regs[0]] = pos

    @staticmethod
    def cost(ln):
        op = ln.split()[0]
        if op == "v_exp_f32":
            return 8
        return 4

    # ---- one step: logits of unit u+1, softmax of unit u, second product of unit u-1.
    # kpre, vpre: read ids of K fragments 0..2 of unit u+1 and V^T fragments 0..2 of unit u-1, already issued.  dma: load
    # instructions to spread over the step (those of the tile whose stage the barrier of the previous step set free).
    # Fragments are read three ahead without a gap between steps.  Even steps hold the barrier of tile u/2: it comes when the
    # last fragment of V of unit u-1 has arrived (nobody reads tile u/2-1 any more) and with the first fragments of tile u/2+1
    # to be read behind it, which are needed after a dozen other matrix instructions.
    def step(self, u, kpre, vpre, dma=()):
        e = self.emit
        with_pv = u > 0
        valu = (self.pending_sums() if u > 0 else []) + self.softmax_all(u % 4) + self.check_list()
        self.check_distances(valu)
        # then the next unit's first key and whether it has to be masked or is none (all of these change the carry bit: one order)
        dma = list(dma) + ["s_add_u32 s66, s66, 32", "s_cmp_ge_i32 s66, s71", "s_cselect_b64 s[64:65], -1, 0"]
        xq, xp = (u + 1) % 4, (u - 1) % 4
        nf = MB * KB                             # fragments of a unit's logits; as many of its second product
        assert nf == DB == 8
        if with_pv:
            slots = [("pv", "ones"), ("pv", 0), ("pv", 1), ("qk", 0), ("qk", 1)]
            for i in range(2, 6):
                slots += [("pv", i), ("qk", i)]
            slots += [("pv", 6), ("qk", 6), ("qk", 7), ("pv", 7)]
        else:
            slots = [("qk", i) for i in range(nf)]
        nsub = QB * len(slots)                   # a slot's matrix instructions share its fragment
        total = sum(self.cost(ln) for ln in valu)
        kids = dict(enumerate(kpre))
        vids = dict(enumerate(vpre))
        next_k, next_v = [], []
        sub = 0
        done_cost = 0
        vi = 0

        for si, (kind, i) in enumerate(slots):
            for n in range(QB):
                qb = QB - 1 - n if si & 1 else n
                if n == 0 and si == 0 and i != "ones":
                    self.wait_for(kids[i] if kind == "qk" else vids[i])
                if kind == "qk":
                    e(self.qk(xq, qb, i, i % 4))
                else:
                    e(self.pv(xp, qb, i))
                # one LDS read or load instruction
                if kind == "qk" and i + 3 < nf:
                    if n == 1:
                        kids[i + 3] = self.k_read(u + 1, i + 3)
                        free = False
                    else:
                        free = True
                elif kind == "qk" and with_pv and (i, n) in ((6, 1), (6, 2), (7, 1)):
                    next_k.append(self.k_read(u + 2, len(next_k)))
                    free = False
                elif kind == "pv" and i != "ones" and n in (1, 2):
                    f = i + 3
                    unit, db = (u - 1, f) if f < nf else (u, f - nf)
                    if n == 1:
                        self.v_read_lo(unit, db)
                    else:
                        rid = self.v_read_hi(unit, db)
                        if f < nf:
                            vids[f] = rid
                        else:
                            next_v.append(rid)
                    free = False
                elif kind == "pv" and i == 6 and n == 0 and not u & 1:
                    free = not self.wait_for(vids[nf - 1])            # V of unit u-1 has been read
                elif kind == "qk" and i == 6 and n == 0 and with_pv and not u & 1:
                    e("s_barrier")
                    free = False
                else:
                    free = True
                if n == QB - 1 and si + 1 < len(slots):
                    # the next fragment is waited for here, where the wait costs nothing if the fragment has arrived
                    assert free
                    k2, i2 = slots[si + 1]
                    free = i2 == "ones" or not self.wait_for(kids[i2] if k2 == "qk" else vids[i2])
                    if kind == "pv" and i == 6 and not u & 1:
                        # tile u/2+1 is published next: this wave's share has landed, all loads but the newest tile's
                        assert free and not dma
                        e(f"s_waitcnt vmcnt({2 * NI})")
                if sub == nsub - 1:
                    assert free and not dma and vi == len(valu)
                    e("s_or_b64 vcc, vcc, s[64:65]")
                    free = False
                if free and dma:
                    e(dma.pop(0))
                sub += 1
                used = 0
                goal = total * sub / (nsub - 2)      # (the outcome of the check is read behind the last one)
                while vi < len(valu):
                    c = self.cost(valu[vi])
                    if sub < nsub - 2 and used + c > CAP and done_cost + c / 2 > goal:
                        break
                    e(valu[vi])
                    done_cost += c
                    used += c
                    vi += 1
        assert vi == len(valu) and not dma
        if not with_pv:
            # the reads ahead, in the order of the other steps
            next_v = [self.v_read(u, 0), self.v_read(u, 1)]
            e(f"s_waitcnt vmcnt({2 * NI})")
            e("s_barrier")
            next_k = [self.k_read(u + 2, f) for f in range(3)]
            next_v.append(self.v_read(u, 2))
        self.finish_sums(u)
        # this wave's share of tile u/2+3 goes out during the step after the barrier
        next_dma = self.dma_list(u // 2 + 3) if u & 1 == 0 else []
        return next_k, next_v, next_dma

    def drain(self, u, vpre):
        """Second product of unit u after the last step, and that unit's sums."""
        e = self.emit
        vids = dict(enumerate(vpre))
        for g in range(DB):
            self.wait_for(vids[g])
            for qb in range(QB):
                e(self.pv(u % 4, qb, g))
            if g + 3 < DB:
                vids[g + 3] = self.v_read(u, g + 3)
        for qb in range(QB):
            e(self.pv(u % 4, qb, "ones"))
        for ln in self.pending_sums():
            e(ln)
        self.emit("s_waitcnt lgkmcnt(0)")      # the K fragments read ahead for a step that does not come
        self.queue = []
        e("s_branch .Lfw64_end_%=")

    def block(self):
        e = self.emit
        for db in range(1, DB):
            e(f"v_xor_b32 {VADDR(db)}, {32 * db}, {VADDR(0)}")
        for tensor in (0, 1):
            for n in range(NI):
                e(f"v_add_u32 {DMAOFF(tensor, n)}, {n * NW * 1024}, {KVOFF if tensor == 0 else VVOFF}")
        e("s_mov_b64 s[60:61], %[kptr]")
        e("s_mov_b64 s[62:63], %[vptr]")
        e("s_lshl_b32 s67, %[ntiles], 6")
        e("s_mov_b32 s69, %[nadvance]")
        e("s_mov_b32 s70, %[maskfrom]")
        e("s_mov_b32 s66, 0")
        e("s_min_i32 s71, s70, s67")
        for r in list(range(128)) + list(range(192, 208)):
            e(f"v_accvgpr_write_b32 a{r}, 0")
        for r in range(168, 172):
            e(f"v_mov_b32 v{r}, {'0x3f803f80' if self.bf16 else '0x3c003c00'}")
        for qb in range(QB):
            e(f"v_mov_b32 {M_REF(qb)}, 0xf149f2ca")    # -1e30
            e(f"v_mov_b32 {L_RUN(qb)}, 0")
        # this wave's share of tile 2 (tiles 0 and 1 were issued, tile 0 published, before the block)
        for ln in self.dma_list(2):
            e(ln)
            e("s_nop 0")
        # logits of unit 0
        ids = [self.k_read(0, f) for f in range(3)]
        for f in range(MB * KB):
            self.wait_for(ids[f])
            for qb in range(QB):
                e(self.qk(0, qb, f, f % 4))
            if f + 3 < MB * KB:
                ids.append(self.k_read(0, f + 3))
        kpre = [self.k_read(1, f) for f in range(3)]
        e("s_nop 15")                               # the first step's vector work reads these logits
        e("s_cmp_lt_i32 s66, s70")
        e("s_cbranch_scc1 .Lfw64_first_%=")
        for ln in self.mask_lines(0, "s66"):
            e(ln)
        e(".Lfw64_first_%=:")
        kpre, vpre, dma = self.step(0, kpre, [])
        e(".Lfw64_loop_%=:")
        entry = [self.labels[q] for q in self.queue]
        state = {}
        for u in range(1, 9):
            kpre, vpre, dma = self.step(u, kpre, vpre, dma=dma)
            if u & 1:
                state[u] = (list(self.queue), vpre)
        assert [self.labels[q] for q in self.queue] == entry and len(entry) == 9
        e("s_branch .Lfw64_loop_%=")
        for u in state:
            e(f".Lfw64_drain_{u}_%=:")
            self.queue, vpre = state[u]
            self.drain(u, vpre)
        self.out += self.cold
        e(".Lfw64_end_%=:")
        e("s_nop 15")      # the accumulators are read by compiler-generated code next
        e("s_nop 3")
        return "\n".join(self.out)


CLOBBER_V = list(range(0, 160)) + list(range(168, 172)) + list(range(174, 181)) + list(range(183, 187)) + list(range(188, 201))
CLOBBER_S = list(range(60, 72))


def generate(path):
    """Writes the generated fragment to `path` (only if its text changes, so that build time stamps stay put)."""
    parts = ["// GENERATED by gen_fa_wide64_loop.py -- do not edit; change the script and build again.",
             "// The software-pipelined check-free main loop of fa_fwd_wide64_kernel as inline assembly with hand-chosen",
             "// registers and instruction order (plan and reasons are in the script's header).  A fragment of fa_fwd.hip.", ""]
    for name, bf16, two_sums in (("FA_WIDE64_LOOP_ASM_F16", False, False), ("FA_WIDE64_LOOP_ASM_F16_TWO_SUMS", False, True),
                                 ("FA_WIDE64_LOOP_ASM_BF16", True, True)):
        parts.append(f"#define {name} \\")
        lines = Gen(bf16, two_sums).block().split("\n")
        parts.append(" \\\n".join('    "' + ln + '\\n\\t"' for ln in lines))
        parts.append("")
    clob = ", ".join([f'"v{r}"' for r in CLOBBER_V] + [f'"s{r}"' for r in CLOBBER_S] + ['"vcc"', '"scc"', '"m0"', '"memory"'])
    parts.append(f"#define FA_WIDE64_LOOP_CLOBBERS {clob}")
    parts.append("")
    text = "\n".join(parts)
    try:
        if open(path).read() == text:
            return
    except OSError:
        pass
    with open(path, "w") as f:
        f.write(text)


if __name__ == "__main__":
    generate(os.path.join(os.path.dirname(os.path.abspath(__file__)), "fa_attention_wide64_loop.inc"))
