#!/usr/bin/env python3
"""Writes pasa_mfma_pipes.hpp: the software-pipelined LDS-read + MFMA sequences of the attention kernel.

Why generated assembly: the operand fetches of an MFMA chain have to be requested several MFMAs ahead of
their use (an LDS read takes longer than an MFMA), which needs a fixed set of operand buffers and counted
waits.  Each sequence is ONE asm statement, so nothing can be scheduled into it and no register of it can
be copied or reused while a read is in flight.  The operand buffers are fixed registers (v226..v255,
declared as clobbered): a transposing read fills half of an MFMA operand, and inline-asm operands cannot
name half of a register tuple.

Run `python gen_mfma_pipes.py` in this directory after changing it; the header is committed.

LDS addressing (see the tile layout in pasa_device.hpp): within a tile, the address of a lane's row
fragment for contraction step s is a0 ^ (s << 5), 32 rows further down is +64*D bytes; the address of a
column fragment of value-column tile t is a0 ^ (t << 6) (and the same for the rows 8 further down, from a
second lane address), 16 rows further down is +32*D bytes.  XOR by a constant and immediate offsets replace
every per-fetch address computation.
"""
import os

FBASE = 232            # operand buffers: 6 x 4 registers v[232:255]
TBASE = 226            # address temporaries v226..v231
CLOBBER_LO, CLOBBER_HI = 226, 255
MFMA = "v_mfma_f32_32x32x16_bf16"
NOP_AFTER = "s_nop 13"  # an 8-pass MFMA result may be read by a VALU instruction 12 wait states later


def F(i):
    return f"v[{FBASE + 4 * i}:{FBASE + 4 * i + 3}]"


def Flo(i):
    return f"v[{FBASE + 4 * i}:{FBASE + 4 * i + 1}]"


def Fhi(i):
    return f"v[{FBASE + 4 * i + 2}:{FBASE + 4 * i + 3}]"


def T(i):
    return f"v{TBASE + i}"


def off(n):
    return f" offset:{n}" if n else ""


def rows_x_q(D, two_halves, dma, waves=4):
    """acc(s) += rowfrag(rows 0..31 [and 32..63], step s) x q[s].
    two_halves: c0 <- rows 0..31, c1 <- rows 32..63.  Otherwise rows 0..31 only, even steps -> c0, odd -> c1.
    dma: number of tile-load instructions per tile of this wave (0 = none); requests a K-like and a V-like
    tile into the slots whose LDS addresses are %[lk], %[lv]."""
    ns = D // 16
    half_off = 64 * D
    frags = []  # (step s, immediate offset, accumulator)
    for s in range(ns):
        if two_halves:
            frags.append((s, 0, "c0"))
            frags.append((s, half_off, "c1"))
        else:
            frags.append((s, 0, "c0" if s % 2 == 0 else "c1"))
    nbuf = 6
    lines = []
    last = {"s": 0, "reg": "%[a]", "n": 0}

    def addr(s):  # LDS instructions read their address when they issue, so a temporary can be reused at once
        if s != last["s"]:
            last["s"], last["reg"] = s, T(last["n"] % 2)
            last["n"] += 1
            lines.append(f"v_xor_b32 {last['reg']}, {hex(s << 5)}, %[a]")
        return last["reg"] if s else "%[a]"

    def issue(i):
        s, o, _ = frags[i]
        lines.append(f"ds_read_b128 {F(i % nbuf)}, {addr(s)}{off(o)}")

    dmas = [("k", j) for j in range(dma)] + [("v", j) for j in range(dma)]
    stride = waves * 1024  # a wave's tile-load instructions are this far apart in LDS
    n = len(frags)
    for i in range(min(nbuf, n)):
        issue(i)
    seen = set()
    for i in range(n):
        outstanding = min(nbuf - 1, n - 1 - i)
        s, _, acc = frags[i]
        lines.append(f"s_waitcnt lgkmcnt({outstanding})")
        src_c = f"%[{acc}]" if acc in seen else "0"
        seen.add(acc)
        lines.append(f"{MFMA} %[{acc}], {F(i % nbuf)}, %[q{s}], {src_c}")
        if dmas:  # in the shadow of the MFMA: one tile-load instruction (M0 = its LDS destination)
            lines.append(f"s_add_u32 m0, %[l{dmas[0][0]}], {hex(dmas[0][1] * stride)}")
        if i + nbuf < n:
            issue(i + nbuf)
        elif dmas:
            lines.append("s_nop 0")  # one wait state between the write of M0 and its use
        if dmas:
            which, jj = dmas.pop(0)
            lines.append(f"global_load_lds_dwordx4 %[x{jj}], %[{which}b]")
    assert not dmas, "more tile-load instructions than MFMAs"
    lines.append(NOP_AFTER)
    return lines


def cols_x_p(D, nks, row0, dma=0):
    """o[t] += colfrag(rows row0 + 16 ks .., value columns 32 t ..) x p[ks], ks < nks, t < D/32.
    dma: as in rows_x_q (two tiles, from %[kb] into the slot at %[lk] and from %[vb] into the slot at %[lv])."""
    nt = D // 32
    step_off = 32 * D
    base_off = row0 * 2 * D
    frags = [(ks, t) for ks in range(nks) for t in range(nt)]
    nbuf = 6
    lines = []
    for t in range(1, nt):  # addresses for t >= 1
        lines.append(f"v_xor_b32 {T(2 * t - 2)}, {hex(t << 6)}, %[a0]")
        lines.append(f"v_xor_b32 {T(2 * t - 1)}, {hex(t << 6)}, %[a1]")

    def a(t, j):
        return (f"%[a{j}]") if t == 0 else T(2 * t - 2 + j)

    def issue(i):
        ks, t = frags[i]
        o = base_off + ks * step_off
        lines.append(f"ds_read_b64_tr_b16 {Flo(i % nbuf)}, {a(t, 0)}{off(o)}")
        lines.append(f"ds_read_b64_tr_b16 {Fhi(i % nbuf)}, {a(t, 1)}{off(o)}")

    dmas = [("k", j) for j in range(dma)] + [("v", j) for j in range(dma)]
    n = len(frags)
    for i in range(min(nbuf, n)):
        issue(i)
    for i in range(n):
        outstanding = 2 * min(nbuf - 1, n - 1 - i)
        ks, t = frags[i]
        lines.append(f"s_waitcnt lgkmcnt({outstanding})")
        lines.append(f"{MFMA} %[o{t}], {F(i % nbuf)}, %[p{ks}], %[o{t}]")
        if dmas:
            lines.append(f"s_add_u32 m0, %[l{dmas[0][0]}], {hex(dmas[0][1] * 4096)}")
        if i + nbuf < n:
            issue(i + nbuf)
        elif dmas:
            lines.append("s_nop 0")
        if dmas:
            which, jj = dmas.pop(0)
            lines.append(f"global_load_lds_dwordx4 %[x{jj}], %[{which}b]")
    assert not dmas, "more tile-load instructions than MFMAs"
    lines.append(NOP_AFTER)
    return lines


# ---- the fused step: logits, online softmax and P V of one 64-key tile whose keys are all valid ----
# The tile is handled as two halves of 32 keys, each with its own online-softmax update, so that the
# VALU work of one half runs in the shadow of the other half's MFMAs (a wave issues a VALU instruction
# only every other issue slot, so a softmax on its own leaves the SIMD mostly idle):
#   S0 = K[0:32] Q^T                      (the next tile pair is requested in the shadow of these MFMAs)
#   S1 = K[32:64] Q^T                     with the softmax of S0 -> P0 in its shadow (accumulators rescaled if needed)
#   O += V[0:32]^T P0                     with the softmax of S1 -> P1 in its shadow
#   (accumulators rescaled if the second half raised the maximum: only now, when no MFMA adds to them)
#   O += V[32:64]^T P1
# Registers.  The accumulators are operands bound to fixed registers (their elements have to be named
# for the rescaling): O v[0:63].  Internal, declared clobbered: S0 v[168:183], S1 v[184:199],
# P0 v[200:207], P1 v[208:215], addresses v[216:223], temporaries v[224:231], operand buffers v[232:255].
FS_O, FS_S0, FS_S1, FS_P0, FS_P1, FS_A, FS_T = 0, 168, 184, 200, 208, 216, 224
FUSED_CLOBBER_LO = 168


def vr(base, n=1):
    return f"v{base}" if n == 1 else f"v[{base}:{base + n - 1}]"


def max_stream(S):
    """T0 = c * max over the lane's 16 logits v[S:S+15]"""
    s = lambda i: vr(S + i)
    t0, t1 = vr(FS_T), vr(FS_T + 1)
    return [f"v_max3_f32 {t0}, {s(0)}, {s(1)}, {s(2)}", f"v_max3_f32 {t1}, {s(8)}, {s(9)}, {s(10)}",
            f"v_max3_f32 {t0}, {t0}, {s(3)}, {s(4)}", f"v_max3_f32 {t1}, {t1}, {s(11)}, {s(12)}",
            f"v_max3_f32 {t0}, {t0}, {s(5)}, {s(6)}", f"v_max3_f32 {t1}, {t1}, {s(13)}, {s(14)}",
            f"v_max3_f32 {t0}, {t0}, {s(7)}, {s(15)}", f"v_max_f32 {t0}, {t0}, {t1}", f"v_mul_f32 {t0}, %[c], {t0}"]


def exp_stream(S, P, convert=True):
    """p = exp2(s c - m) in place, the two P^T fragments into v[P:P+7] (if convert), l += sum.  Three-stage
    pipeline so that no instruction uses the result of the transcendental issued right before it."""
    s = lambda i: vr(S + i)
    t4 = vr(FS_T + 4)
    out = []
    for i in range(19):
        if i < 16:
            out.append(f"v_fma_f32 {s(i)}, {s(i)}, %[c], -%[m]")
        if 1 <= i <= 16:
            out.append(f"v_exp_f32 {s(i - 1)}, {s(i - 1)}")
        e = i - 3
        if 0 <= e < 16:
            if e % 2 == 0:
                out.append(f"v_add_f32 %[l], %[l], {s(e)}")
            elif e == 3:
                out.append(f"v_add_f32 {t4}, {s(1)}, {s(3)}")
            elif e > 3:
                out.append(f"v_add_f32 {t4}, {t4}, {s(e)}")
            if e % 2 == 1 and convert:
                out.append(f"v_cvt_pk_bf16_f32 {vr(P + e // 2)}, {s(e - 1)}, {s(e)}")
    out.append(f"v_add_f32 %[l], %[l], {t4}")
    return out


def convert_stream(S, P):
    return [f"v_cvt_pk_bf16_f32 {vr(P + j)}, {vr(S + 2 * j)}, {vr(S + 2 * j + 1)}" for j in range(8)]


def raise_max(n_o, now, also=()):
    """after max_stream: if the maximum grew for some lane, m <- max(m, T0 of both lanes of the query), T3 = exp2(m_old - m),
    l *= T3, and either the accumulators too (now) or the wave-uniform decision is left in %[flag] for later.
    The lane's own maximum decides: both lanes of a query hold the same m, so one of them sees the growth, and the exchange
    with lane ^ 32 (four instructions and their wait states in the middle of a dependence chain) is only made then, in about
    every fourth half.
    The conditional part is one item: it must not be split up (nothing else may sit between branch and label)."""
    t0, t1, t2, t3 = (vr(FS_T + i) for i in range(4))
    tag = "a" if now else "b"
    out = [f"v_cmp_gt_f32 vcc, {t0}, %[m]"]
    if not now:
        out.append("s_mov_b64 %[flag], vcc")
    cond = [f"s_cbranch_vccz .Lfs_keep{tag}_%=",
            f"v_mov_b32 {t1}, {t0}", "s_nop 1", f"v_permlane32_swap_b32 {t0}, {t1}", "s_nop 0",
            f"v_max3_f32 {t1}, %[m], {t0}, {t1}", f"v_sub_f32 {t2}, %[m], {t1}", f"v_exp_f32 {t3}, {t2}",
            f"v_mov_b32 %[m], {t1}", "s_nop 0", f"v_mul_f32 %[l], %[l], {t3}"]
    if now:
        cond += [f"v_mul_f32 {vr(FS_O + i)}, {vr(FS_O + i)}, {t3}" for i in range(n_o)]
    cond += [f"v_mul_f32 {r}, {r}, {t3}" for r in also]  # e.g. weights computed against the old maximum, not yet used
    cond.append(f".Lfs_keep{tag}_%=:")
    out.append(tuple(cond))
    return out


class LdsPipe:
    """fragment loads into the ring of operand buffers, with the bookkeeping for counted waits"""
    def __init__(self, lines, D, nbuf=6):
        self.lines, self.D, self.nbuf, self.issued, self.v_ready = lines, D, nbuf, [], False

    def k_addresses(self):
        for st in range(1, self.D // 16):
            self.lines.append(f"v_xor_b32 {vr(FS_A + st - 1)}, {hex(st << 5)}, %[ak]")

    def v_addresses(self):
        for t in range(1, self.D // 32):
            self.lines.append(f"v_xor_b32 {vr(FS_A + 2 * t - 2)}, {hex(t << 6)}, %[av0]")
            self.lines.append(f"v_xor_b32 {vr(FS_A + 2 * t - 1)}, {hex(t << 6)}, %[av1]")
        self.v_ready = True

    def issue(self, k, load):
        f = k % self.nbuf
        kind, a, b = load
        if kind == "k":
            st, half = a, b
            addr = "%[ak]" if st == 0 else vr(FS_A + st - 1)
            self.lines.append(f"ds_read_b128 {F(f)}, {addr}{off(half * 64 * self.D)}")
            self.issued.append(1)
        else:
            if not self.v_ready:  # all K reads have been issued by now: their address registers are free
                self.v_addresses()
            ks, t = a, b
            a0 = "%[av0]" if t == 0 else vr(FS_A + 2 * t - 2)
            a1 = "%[av1]" if t == 0 else vr(FS_A + 2 * t - 1)
            self.lines.append(f"ds_read_b64_tr_b16 {Flo(f)}, {a0}{off(ks * 32 * self.D)}")
            self.lines.append(f"ds_read_b64_tr_b16 {Fhi(f)}, {a1}{off(ks * 32 * self.D)}")
            self.issued.append(2)

    def wait_for(self, k):
        outstanding = sum(self.issued[k + 1:])
        assert outstanding <= 15
        self.lines.append(f"s_waitcnt lgkmcnt({outstanding})")


def spread(after, k0, k1, stream):
    """distributes the items of `stream` over the slots k0..k1 (instructions that follow MFMA k); an item that
    is a tuple of instructions stays together"""
    nslots = k1 - k0 + 1
    per = -(-len(stream) // nslots)
    for i in range(nslots):
        for item in stream[i * per:(i + 1) * per]:
            after.setdefault(k0 + i, []).extend(list(item) if isinstance(item, tuple) else [item])


def fused_step(D, waves):
    ns, nt = D // 16, D // 32
    ni = tile_loads(D, waves)
    n_o = 16 * nt
    mf = []
    for half in range(2):
        for st in range(ns):
            mf.append(dict(acc=vr(FS_S0 if half == 0 else FS_S1, 16), first=(st == 0), b=f"%[q{st}]", load=("k", st, half)))
    for half in range(2):
        for ks2 in range(2):
            for t in range(nt):
                mf.append(dict(acc=vr(FS_O + 16 * t, 16), first=False, b=vr((FS_P0 if half == 0 else FS_P1) + 4 * ks2, 4),
                               load=("v", 2 * half + ks2, t)))
    n = len(mf)
    after = {}
    qk1_end, pv0_end = 2 * ns - 1, 2 * ns + 2 * nt - 1
    spread(after, ns + 1, qk1_end, max_stream(FS_S0) + raise_max(n_o, True) + exp_stream(FS_S0, FS_P0))
    spread(after, 2 * ns + 1, pv0_end, max_stream(FS_S1) + raise_max(n_o, False) + exp_stream(FS_S1, FS_P1))
    # the accumulators are rescaled for the second half once the MFMAs that add to them are done
    after[pv0_end] += ["s_cmp_eq_u64 %[flag], 0", "s_cbranch_scc1 .Lfs_nors_%=", "s_nop 13"] + \
        [f"v_mul_f32 {vr(FS_O + i)}, {vr(FS_O + i)}, {vr(FS_T + 3)}" for i in range(n_o)] + [".Lfs_nors_%=:"]
    before = {2 * ns: ["s_nop 1"], 2 * ns + 2 * nt: ["s_nop 1"]}  # P^T / accumulators were written by VALU just before

    lines = []
    pipe = LdsPipe(lines, D)
    pipe.k_addresses()
    for k in range(pipe.nbuf):
        pipe.issue(k, mf[k]["load"])
    dmas = [("k", j) for j in range(ni)] + [("v", j) for j in range(ni)]
    for k in range(n):
        pipe.wait_for(k)
        lines += before.get(k, [])
        m = mf[k]
        lines.append(f"{MFMA} {m['acc']}, {F(k % pipe.nbuf)}, {m['b']}, {'0' if m['first'] else m['acc']}")
        if dmas:
            lines.append(f"s_add_u32 m0, %[l{dmas[0][0]}], {hex(dmas[0][1] * waves * 1024)}")
        if k + pipe.nbuf < n:
            pipe.issue(k + pipe.nbuf, mf[k + pipe.nbuf]["load"])
        elif dmas:
            lines.append("s_nop 0")
        if dmas:
            which, jj = dmas.pop(0)
            lines.append(f"global_load_lds_dwordx4 %[x{jj}], %[{which}b]")
        lines += after.get(k, [])
    assert not dmas
    lines.append(NOP_AFTER)
    return lines


# ---- the pipelined step: the same work, with the logits one tile ahead of P V ----
# In the chain logits -> maximum -> exponentials -> P V of one tile only the matrix work of OTHER keys can run beside the
# softmax.  So a step takes P V of tile t and the logits of tile t + 1, and the softmax in between has MFMAs on both sides
# that do not wait for it.  Half h = 32 keys; on entry P(2t) is ready and the logits of half 2t + 1 are complete:
#   logits of half 2t + 2 -> S0,  O += V[0:32]^T P(2t),        softmax of half 2t + 1: S1 -> P1
#   logits of half 2t + 3 -> S1,  O += V[32:64]^T P(2t + 1),   softmax of half 2t + 2: S0 -> P0
# The vector instructions (about 680 cycles of issue at 4 each, 8 for an exponential) are spread evenly over the shadows of
# the 32 MFMAs (32 cycles each, of which they leave 24 for other vector instructions).
# A half that raises the maximum leaves the factor for the accumulators: it is applied after the P V of the half
# before it, in the shadow of the logits that follow; the second half's is handed to the next step (corr, flag).  The rare blocks
# (.subsection) lie behind the kernel, so the usual way has no taken branch in it.
# LDS: the ring's K slots are 0 and 2, the V slots 1 and 3; a step of parity `par` reads V from slot 2 par + 1 and K from
# the other K slot, so every fetch is a lane address that stays the same for all tiles plus an immediate offset.
class Cold:
    """blocks that are jumped to and from, kept out of the instruction stream"""
    def __init__(self, prefix):
        self.prefix, self.n, self.lines = prefix, 0, []

    def block(self, branch, body):
        """-> instructions that run `body` if `branch` jumps"""
        t = f".L{self.prefix}{self.n}"
        self.n += 1
        self.lines += [f"{t}_%=:"] + body + [f"s_branch {t}r_%="]
        return [f"{branch} {t}_%=", f"{t}r_%=:"]

    def text(self):
        return [".subsection 1"] + self.lines + [".subsection 0"] if self.lines else []


def growth(cold, flag, corr, also=()):
    """after max_stream: where the maximum grew for some lane, m, l and the factor `corr` for the accumulators; `flag` is not
    zero then (without a flag: corr is 1 where there is nothing to do).  (The lane's own maximum decides, see raise_max.)"""
    t0, t1, t2 = (vr(FS_T + i) for i in range(3))
    body = [f"v_mov_b32 {t1}, {t0}", "s_nop 1", f"v_permlane32_swap_b32 {t0}, {t1}", "s_nop 0",
            f"v_max3_f32 {t1}, %[m], {t0}, {t1}", f"v_sub_f32 {t2}, %[m], {t1}", f"v_exp_f32 {corr}, {t2}",
            f"v_mov_b32 %[m], {t1}", "s_nop 0", f"v_mul_f32 %[l], %[l], {corr}"] + [f"v_mul_f32 {r}, {r}, {corr}" for r in also]
    note = f"s_mov_b64 {flag}, vcc" if flag else f"v_mov_b32 {corr}, 1.0"
    return tuple([f"v_cmp_gt_f32 vcc, {t0}, %[m]", note] + cold.block("s_cbranch_vccnz", body))


def pending(cold, flag, corr, n_o, nop):
    """accumulators *= corr if flag is not zero (without a flag: if corr is not 1 in some lane)"""
    test = [f"s_cmp_lg_u64 {flag}, 0"] if flag else [f"v_cmp_neq_f32 vcc, 1.0, {corr}"]
    return tuple(test + cold.block("s_cbranch_scc1" if flag else "s_cbranch_vccnz", [nop] + [f"v_mul_f32 {vr(FS_O + i)}, {vr(FS_O + i)}, {corr}" for i in range(n_o)]))


def cost(item):
    if isinstance(item, tuple):
        return 8
    return 8 if item.startswith("v_exp") else 4


def pour(after, n_slots, stream, first=0, begin=0.0, end=1.0):
    """distributes the items of `stream` over the slots so that the issue cycles grow linearly from slot begin * n_slots
    to end * n_slots"""
    total = sum(cost(x) for x in stream)
    done = 0
    for item in stream:
        k = int((begin + (end - begin) * done / total) * n_slots)
        after.setdefault(max(first, min(k, n_slots - 1)), []).extend(list(item) if isinstance(item, tuple) else [item])
        done += cost(item)


def pipe_run(D, mf, before, after, dmas, cold, par, prologue=(), waves=4):
    """MFMA k of `mf` with its operand fetch issued six MFMAs ahead (load: ("k", step, half) from the K slot, ("v", 16-row
    step, column tile) from the V slot)"""
    lines, issued, nbuf = [], [], 6
    k_off, v_off = (1 - par) * 128 * D * 2, par * 128 * D * 2

    def issue(k):
        f = k % nbuf
        kind, a, b = mf[k]["load"]
        if kind == "k":
            lines.append(f"ds_read_b128 {F(f)}, %[ka{a}]{off(k_off + b * 64 * D)}")
            issued.append(1)
        else:
            lines.append(f"ds_read_b64_tr_b16 {Flo(f)}, %[va{2 * b}]{off(v_off + a * 32 * D)}")
            lines.append(f"ds_read_b64_tr_b16 {Fhi(f)}, %[va{2 * b + 1}]{off(v_off + a * 32 * D)}")
            issued.append(2)

    n = len(mf)
    for k in range(min(nbuf, n)):
        issue(k)
    lines += list(prologue)
    dmas = list(dmas)
    for k in range(n):
        outstanding = sum(issued[k + 1:])
        assert outstanding <= 15
        lines.append(f"s_waitcnt lgkmcnt({outstanding})")
        lines += before.get(k, [])
        m = mf[k]
        lines.append(f"{MFMA} {m['acc']}, {F(k % nbuf)}, {m['b']}, {'0' if m['first'] else m['acc']}")
        if dmas:
            lines.append(f"s_add_u32 m0, %[l{dmas[0][0]}], {hex(dmas[0][1] * waves * 1024)}")
        if k + nbuf < n:
            issue(k + nbuf)
        elif dmas:
            lines.append("s_nop 0")
        if dmas:
            which, jj = dmas.pop(0)
            lines.append(f"global_load_lds_dwordx4 %[x{jj}], %[{which}b]")
        lines += after.get(k, [])
    assert not dmas
    return lines


def qk_mfmas(D, half):
    return [dict(acc=vr(FS_S0 if half == 0 else FS_S1, 16), first=(st == 0), b=f"%[q{st}]", load=("k", st, half)) for st in range(D // 16)]


def pv_mfmas(D, half):
    return [dict(acc=vr(FS_O + 16 * t, 16), first=False, b=vr((FS_P0 if half == 0 else FS_P1) + 4 * ks2, 4), load=("v", 2 * half + ks2, t))
            for ks2 in range(2) for t in range(D // 32)]


def tile_loads(D, waves):
    """tile-load instructions of one wave"""
    return D // 8 // waves


def pipe_step(D, par, waves):
    nt = D // 32
    ni = tile_loads(D, waves)
    n_o = 16 * nt
    mf = qk_mfmas(D, 0) + pv_mfmas(D, 0) + qk_mfmas(D, 1) + pv_mfmas(D, 1)
    n, q = len(mf), len(mf) // 4
    cold = Cold(f"ps{par}_")
    corr1 = vr(FS_T + 3)
    after = {}
    after[1] = list(pending(cold, "%[flag]", "%[corr]", n_o, "s_nop 3"))  # left by the step before
    # (done with S1 before the MFMAs of the second half write it; S0 is long complete)
    pour(after, n, [growth(cold, "%[flag1]", corr1)] + exp_stream(FS_S1, FS_P1), first=1, end=0.5)
    pour(after, n, max_stream(FS_S0) + [growth(cold, "%[flag]", "%[corr]")] + exp_stream(FS_S0, FS_P0), begin=0.5)
    k = 2 * q + 1  # the P V of half 2t is through
    after[k] = list(pending(cold, "%[flag1]", corr1, n_o, "s_nop 3")) + after.get(k, [])
    dmas = [("k", j) for j in range(ni)] + [("v", j) for j in range(ni)]
    lines = pipe_run(D, mf, {}, after, dmas, cold, par, prologue=max_stream(FS_S1), waves=waves)
    return lines + cold.text()


def pipe_start(D):
    """logits of the first tile (K slot 0) and the softmax of its first half"""
    mf = qk_mfmas(D, 0) + qk_mfmas(D, 1)
    n, q = len(mf), len(mf) // 2
    cold = Cold("pb")
    after = {}
    pour(after, n, max_stream(FS_S0) + [growth(cold, "%[flag]", "%[corr]")] + exp_stream(FS_S0, FS_P0), first=q + 1, begin=(q + 1) / n)
    return pipe_run(D, mf, {}, after, [], cold, 1) + [NOP_AFTER] + cold.text()


def pipe_end(D, par):
    """P V of the last tile (V slot 2 par + 1) and the softmax of its second half"""
    n_o = 16 * (D // 32)
    mf = pv_mfmas(D, 0) + pv_mfmas(D, 1)
    n, q = len(mf), len(mf) // 2
    cold = Cold(f"pe{par}_")
    after = {}
    pour(after, q, [growth(cold, "%[flag]", "%[corr]")] + exp_stream(FS_S1, FS_P1))
    before = {q: list(pending(cold, "%[flag]", "%[corr]", n_o, NOP_AFTER)) + ["s_nop 1"]}
    lines = pipe_run(D, mf, before, after, [], cold, par,
                     prologue=list(pending(cold, "%[flag]", "%[corr]", n_o, NOP_AFTER)) + max_stream(FS_S1) + ["s_nop 1"])
    return lines + [NOP_AFTER] + cold.text()


def both_parities(name, make):
    """one statement for the two parities: the compiler keeps the fixed registers in place over a loop around one statement"""
    return [f"s_cmp_lg_u32 %[par], 0", f"s_cbranch_scc1 .L{name}odd_%="] + make(0) + [f"s_branch .L{name}done_%=", f".L{name}odd_%=:"] + \
        make(1) + [f".L{name}done_%=:"]


def pipe_functions():
    out = []
    clobber = lambda regs: ", ".join([f'"v{r}"' for r in regs] + ['"memory"', '"scc"', '"vcc"', '"m0"'])
    s0, p1, rest = range(FS_S0, FS_S0 + 16), range(FS_P1, FS_P1 + 8), list(range(FS_T, 256))
    for D in (128, 64):
        ns, nt = D // 16, D // 32
        state = (f"f32x16 (&o)[{nt}], float& m, float& l, PipeState& st")
        ml = ['[m] "+v"(m)', '[l] "+v"(l)']
        sb = '"+{v[184:199]}"(st.s1)'
        pa = [f'"+{{v[{200 + 4 * k}:{203 + 4 * k}]}}"(st.p0[{k}])' for k in range(2)]
        carry = ['[corr] "+v"(st.corr)', '[flag] "+s"(st.flag)']
        kin = [f'[ka{s}] "v"(ka[{s}])' for s in range(ns)] + q_inputs(D)
        vin = [f'[va{s}] "v"(va[{s}])' for s in range(2 * nt)]
        cin = ['[c] "s"(c)']
        dma = lambda ni: ['[kb] "s"(kb)', '[vb] "s"(vb)', '[lk] "s"(lk)', '[lv] "s"(lv)'] + [f'[x{j}] "v"(x[{j}])' for j in range(ni)]

        def emit(comment, head, pre, lines, outs, ins, clob):
            text = "\n".join(f'      "{l}\\n\\t"' for l in lines)
            out.append(f"{comment}PASA_DEVICE void {head} {{\n{pre}  asm volatile(\n{text}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n"
                       f"      : {clobber(clob)});\n}}\n\n")

        emit("// Start of a run of pipelined steps: logits of the tile in K slot 0, softmax of its first half.  ka, va: the lane's addresses of\n"
             "// the row fragments in K slot 0 and of the column fragments in V slot 1; corr, flag of the state are outputs.\n",
             f"pipe_start(const uint32_t (&ka)[{ns}], const bf16x8 (&q)[{ns}], float& m, float& l, float c, PipeState& st)", "",
             pipe_start(D), ml + ['"=&{v[184:199]}"(st.s1)'] + [x.replace("+", "=&") for x in pa] + ['[corr] "=&v"(st.corr)', '[flag] "=&s"(st.flag)'],
             kin + cin, list(s0) + list(range(FS_P1, FS_P1 + 8)) + rest)
        par_in = ['[par] "s"(par)']
        for waves in (4, 8):
            ni = tile_loads(D, waves)
            emit(f"// P V of the tile in V slot 2 par + 1, logits of the next one, in K slot 2 - 2 par; two more tiles are requested (see\n"
                 f"// rows_x_q_dma) by the {waves} waves of the workgroup.\n",
                 f"pipe_step(int par, const uint32_t (&ka)[{ns}], const uint32_t (&va)[{2 * nt}], const bf16x8 (&q)[{ns}], {state}, float c,\n"
                 f"                          const void* kb, const void* vb, const uint32_t (&x)[{ni}], uint32_t lk, uint32_t lv)",
                 "  uint64_t flag1;\n", both_parities("ps", lambda par: pipe_step(D, par, waves)),
                 o_ops(nt) + ml + [sb] + pa + carry + ['[flag1] "=&s"(flag1)'], kin + vin + cin + dma(ni) + par_in, list(s0) + list(p1) + rest)
        emit("// End of a run: P V of the tile in V slot 2 par + 1.\n",
             f"pipe_end(int par, const uint32_t (&va)[{2 * nt}], {state}, float c)", "", both_parities("pe", lambda par: pipe_end(D, par)),
             o_ops(nt) + ml + [sb] + pa + carry, vin + cin + par_in, list(s0) + list(p1) + rest)
    return "".join(out)


# ---- half of a pipelined step, for workgroups whose groups of waves work on tiles of their own (quad passes, d = 128) ----
# Half `par` of a step: logits of 32 keys of the group's next tile -> S[par], P V of 32 keys of its current tile with P[par], and the
# softmax of S[1 - par] -> P[1 - par] in between.  A run of steps starts with P[0], S[1] of its first tile (quad_start0/1) and ends
# with P V alone (quad_end0/1, which leave nothing pending).  sk, sv: LDS addresses of the group's K and V half slots; kl, vl: the
# lane's offsets of the fragments in a half slot.
# Layout of a half slot: blocks of four rows (one tile-load instruction), padded by 16 bytes so that the four blocks that
# a row fragment touches in one go start four banks apart; inside a row the 16-byte chunk c lies at c ^ ((row & 3) << 2).  So the
# contraction steps 2 j and 2 j + 1 of a row fragment are 32 bytes apart and a column fragment's rows further down an immediate
# offset away: four lane addresses each (eight additions per half step instead of sixteen).
QUAD_BLOCK = 1040               # bytes of a padded block of four rows
QUAD_HALF = 8 * QUAD_BLOCK
QUAD_SLOTS = 18                 # half slots of the ring
QUAD_D = 128


QUAD_RUNS = ((1, 1), (2, 2), (3, 1), (4, 1), (3, 3), (4, 4))  # tiles of even and odd steps


def quad_depth(width):
    """batches of `width` half tiles that the ring holds"""
    return QUAD_SLOTS // width


def quad_loads(kind, a, t, f):
    """instructions that fetch MFMA operand f: row fragment of step a ("k"), column fragment of 16-row step a, column tile t ("v")"""
    if kind == "k":
        return [f"ds_read_b128 {F(f)}, {vr(FS_A + a // 2)}{off(32 * (a % 2))}"]
    return [f"ds_read_b64_tr_b16 {Flo(f)}, {vr(FS_A + 4 + t)}{off(4 * QUAD_BLOCK * a)}",
            f"ds_read_b64_tr_b16 {Fhi(f)}, {vr(FS_A + 4 + t)}{off(4 * QUAD_BLOCK * a + 2 * QUAD_BLOCK)}"]


def quad_run(mf, before, after, prologue, dmas=(), early=()):
    """dmas: (operand of the lane offsets, operand of the base, LDS offset), in the shadows from the second MFMA on; early: instructions
    before the fragment fetches (LDS reads among them have landed by the first MFMA)"""
    lines, issued, nbuf = list(early), [], 6
    kinds = {m["load"][0] for m in mf}
    if "k" in kinds:
        lines += [f"v_add_u32 {vr(FS_A + j)}, %[sk], %[kl{j}]" for j in range(4)]
    if "v" in kinds:
        lines += [f"v_add_u32 {vr(FS_A + 4 + j)}, %[sv], %[vl{j}]" for j in range(4)]

    def issue(k):
        ls = quad_loads(*mf[k]["load"], k % nbuf)
        lines.extend(ls)
        issued.append(len(ls))

    dmas = list(dmas)
    n = len(mf)
    for k in range(min(nbuf, n)):
        issue(k)
    lines += list(prologue)
    for k in range(n):
        outstanding = sum(issued[k + 1:])
        assert outstanding <= 15
        lines.append(f"s_waitcnt lgkmcnt({outstanding})")
        lines += before.get(k, [])
        m = mf[k]
        lines.append(f"{MFMA} {m['acc']}, {F(k % nbuf)}, {m['b']}, {'0' if m['first'] else m['acc']}")
        load = dmas.pop(0) if dmas and k > 0 else None
        if load:
            lines.append(f"s_add_u32 m0, %[ld], {hex(load[2])}")
        if k + nbuf < n:
            issue(k + nbuf)
        elif load:
            lines.append("s_nop 0")
        if load:
            lines.append(f"global_load_lds_dwordx4 {load[0]}, {load[1]}")
        lines += after.get(k, [])
    assert not dmas
    return lines


def quad_parts(par):
    D = QUAD_D
    ns, nt = D // 16, D // 32
    Sx, Sy = (FS_S0, FS_S1) if par == 0 else (FS_S1, FS_S0)
    Px, Py = (FS_P0, FS_P1) if par == 0 else (FS_P1, FS_P0)
    qk = [dict(acc=vr(Sx, 16), first=(st == 0), b=f"%[q{st}]", load=("k", st, 0)) for st in range(ns)]
    pv = [dict(acc=vr(FS_O + 16 * t, 16), first=False, b=vr(Px + 4 * ks, 4), load=("v", ks, t)) for ks in range(2) for t in range(nt)]
    grow = lambda cold: growth(cold, None, "%[corr]")
    pend = lambda cold, nop: list(pending(cold, None, "%[corr]", 16 * nt, nop))
    return qk, pv, Sy, Py, grow, pend


def quad_both(cold, par, dmas=(), early=(), first=()):
    """first: instructions in the shadow of the first MFMA"""
    qk, pv, Sy, Py, grow, pend = quad_parts(par)
    after = {0: list(first), 1: pend(cold, "s_nop 3")}
    pour(after, len(qk + pv), [grow(cold)] + exp_stream(Sy, Py), first=1)
    return quad_run(qk + pv, {}, after, max_stream(Sy), dmas, early)


def quad_steady(kind, cold):
    """steps of a run with na and nb tiles in turn, %[count] > 0 times one (na = nb) or two of them.  A half step of half p requests the
    batch depth - 1 further on, which belongs to half p of its step if depth is odd and to the other half if it is even; the
    tiles of a step (byte offsets xk, those of the step before in xv) come from the step list (lane address la) when its
    half 0 is requested.  ko, vo: where in a batch the group's K and V half tiles lie; for the step after the next they come from the list's
    group bits (lane address lc) in half 1: one tile is everybody's, of four every group has the one with its number."""
    na, nb = QUAD_RUNS[kind]
    width = na + nb
    depth, batch = quad_depth(width), width * QUAD_HALF
    lead = depth - 1
    n_of = lambda t: (na, nb)[t % 2]
    lines = [f".Lqt{kind}_%=:"]
    for s in range(1 if na == nb else 2):  # step s: P V of its tiles, logits of step s + 1
        for par in range(2):
            half, tr = (par + lead) % 2, s + 1 + (par + lead) // 2  # the requested batch: K of step tr, V of step tr - 1
            nk, nv = n_of(tr), n_of(tr - 1)
            lines += [f"s_waitcnt vmcnt({(depth - 2) * width}) lgkmcnt(0)", "s_barrier", "s_add_u32 %[sk], %[sb], %[ko]", "s_add_u32 %[sv], %[sb], %[vo]"]
            early, first = [], []
            if half == 0:
                early += [f"ds_read_u16 %[w{j}], %[la]{off(2 * j)}" for j in range(nk)]
                first += [f"v_mov_b32 %[xv{j}], %[xk{j}]" for j in range(nv)]
                for j in range(nk):
                    first += [f"v_and_b32 %[w{j}], 0xfff, %[w{j}]", f"v_mul_lo_u32 %[w{j}], %[w{j}], %[tb]"]
                first += [f"v_add_u32 %[xk{j}], %[x], %[w{j}]" for j in range(nk)] + [f"v_add_u32 %[la], {2 * nk}, %[la]"]
            n2 = n_of(s + 2)
            if par == 1:
                if n2 in (2, 3):
                    early += [f"ds_read_u16 %[e{j}], %[lc]{off(2 * j)}" for j in range(n2 - 1)]
                    first += [f"v_readfirstlane_b32 %[u{j}], %[e{j}]" for j in range(n2 - 1)] + [f"v_add_u32 %[lc], {2 * (n2 + (n_of(s + 3) if na != nb else 0))}, %[lc]"]
                    if n2 == 3:
                        first += ["s_bitcmp1_b32 %[u1], %[bit]", "s_cselect_b32 %[u1], 1, 2", f"s_mul_i32 %[u1], %[u1], {QUAD_HALF}"]
                    else:
                        first += [f"s_movk_i32 %[u1], {QUAD_HALF}"]
                    first += ["s_bitcmp1_b32 %[u0], %[bit]", "s_cselect_b32 %[u0], 0, %[u1]"]
                else:
                    first += ["s_mov_b32 %[u0], 0" if n2 == 1 else "s_mov_b32 %[u0], %[go]"]
            dmas = [(f"%[xk{j}]", f"%[kb{half}]", j * QUAD_HALF) for j in range(nk)] + \
                   [(f"%[xv{j}]", f"%[vb{half}]", (nk + j) * QUAD_HALF) for j in range(nv)]
            stream = quad_both(cold, par, dmas, early, first)
            # the next batch, and the slot of this one for the next request
            lines += stream + [f"s_add_u32 %[ld], %[sb], %[wp]", f"s_add_u32 %[sb], %[sb], {batch}", f"s_cmp_eq_u32 %[sb], %[end]",
                               f"s_cselect_b32 %[sb], %[ring], %[sb]"]
            if par == 1:
                lines += [f"s_add_u32 %[vo], %[ko], {n2 * QUAD_HALF}", "s_mov_b32 %[ko], %[u0]"]
    return lines + ["s_sub_u32 %[count], %[count], 1", "s_cmp_lg_u32 %[count], 0", f"s_cbranch_scc1 .Lqt{kind}_%="]


def quad_all_steady():
    cold = Cold("qy")
    lines = ["s_cmp_eq_u32 %[count], 0", "s_cbranch_scc1 .Lqtdone_%="]
    for kind in range(len(QUAD_RUNS)):
        lines += [f"s_cmp_lg_u32 %[kind], {kind}", f"s_cbranch_scc1 .Lqtnot{kind}_%="] + quad_steady(kind, cold) + ["s_branch .Lqtdone_%=", f".Lqtnot{kind}_%=:"]
    return lines + [".Lqtdone_%=:"] + cold.text()


def quad_if_active(tag, lines):
    return ["s_cmp_eq_u32 %[active], 0", f"s_cbranch_scc1 .L{tag}skip_%="] + lines + [f".L{tag}skip_%=:"]


def quad_start(par):
    qk, pv, Sy, Py, grow, pend = quad_parts(par)
    if par == 0:
        return quad_if_active("qs0", quad_run(qk, {}, {}, []) + [NOP_AFTER])
    cold = Cold("qs")
    after = {}
    pour(after, len(qk), [grow(cold)] + exp_stream(Sy, Py))
    return quad_if_active("qs1", quad_run(qk, {}, after, max_stream(Sy)) + [NOP_AFTER]) + cold.text()


def quad_plain(par):
    cold = Cold(f"qb{par}")
    return quad_if_active(f"qb{par}", quad_both(cold, par)) + cold.text()


def quad_end(par):
    qk, pv, Sy, Py, grow, pend = quad_parts(par)
    cold = Cold(f"qe{par}")
    after = {}
    if par == 0:
        pour(after, len(pv), [grow(cold)] + exp_stream(Sy, Py))
        lines = quad_run(pv, {}, after, pend(cold, NOP_AFTER) + max_stream(Sy) + ["s_nop 1"])
    else:
        lines = quad_run(pv, {}, {}, pend(cold, NOP_AFTER) + ["s_nop 1"])
    return quad_if_active(f"qe{par}", lines + [NOP_AFTER]) + cold.text()


def quad_functions():
    D = QUAD_D
    ns, nt = D // 16, D // 32
    out = ["// What the half steps of the quad passes hand on (see PipeState).\n"
           "struct QuadState {\n  f32x16 s0, s1;\n  bf16x8 p0[2], p1[2];\n  float corr;  // factor the accumulators still have to be multiplied by\n};\n\n"
           f"constexpr int kQuadBlock = {QUAD_BLOCK};  // bytes of a padded block of four rows of a half slot\n"
           f"constexpr int kQuadSlots = {QUAD_SLOTS};  // half slots of the ring\n"
           f"constexpr int kQuadKinds = {len(QUAD_RUNS)};  // kinds of runs: tiles of their even and odd steps\n"
           f"constexpr int kQuadEven[] = {{{', '.join(str(r[0]) for r in QUAD_RUNS)}}}, kQuadOdd[] = {{{', '.join(str(r[1]) for r in QUAD_RUNS)}}};\n\n"]
    all_state = ['"+{v[168:183]}"(st.s0)', '"+{v[184:199]}"(st.s1)'] + [f'"+{{v[{200 + 4 * k}:{203 + 4 * k}]}}"(st.p0[{k}])' for k in range(2)] + \
        [f'"+{{v[{208 + 4 * k}:{211 + 4 * k}]}}"(st.p1[{k}])' for k in range(2)] + ['[corr] "+v"(st.corr)']
    kin = [f'[kl{j}] "v"(kl[{j}])' for j in range(4)] + q_inputs(D)
    vin = [f'[vl{j}] "v"(vl[{j}])' for j in range(4)]
    cin, skin, svin, act = ['[c] "s"(c)'], ['[sk] "s"(sk)'], ['[sv] "s"(sv)'], ['[active] "s"(active)']
    ml = ['[m] "+v"(m)', '[l] "+v"(l)']
    clob = ", ".join([f'"v{r}"' for r in range(FS_A, 256)] + ['"memory"', '"scc"', '"vcc"', '"m0"'])
    qargs = f"const uint32_t (&kl)[4], const bf16x8 (&q)[{ns}]"
    oargs = f"f32x16 (&o)[{nt}], float& m, float& l, QuadState& st, float c"

    def emit(comment, head, pre, lines, outs, ins):
        text = "\n".join(f'      "{l}\\n\\t"' for l in lines)
        out.append(f"{comment}PASA_DEVICE void {head} {{\n{pre}  asm volatile(\n{text}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n"
                   f"      : {clob});\n}}\n\n")

    for par in range(2):
        emit(f"// First step of a run, half {par} (active = 0: nothing).\n",
             f"quad_start{par}(int active, uint32_t sk, {qargs}, float& m, float& l, QuadState& st, float c)", "",
             quad_start(par), ml + all_state, kin + cin + skin + act)
        emit(f"// Step of a run, half {par} (active = 0: nothing).\n",
             f"quad_half{par}(int active, uint32_t sk, uint32_t sv, {qargs}, const uint32_t (&vl)[4], {oargs})", "",
             quad_plain(par), o_ops(nt) + ml + all_state, kin + vin + cin + skin + svin + act)
        emit(f"// Last step of a run, half {par} (active = 0: nothing).\n", f"quad_end{par}(int active, uint32_t sv, const uint32_t (&vl)[4], {oargs})", "",
             quad_end(par), o_ops(nt) + ml + all_state, vin + cin + svin + act)
    tiles = [f'[{w}{j}] "+v"(t.{w}[{j}])' for w in ("xk", "xv") for j in range(4)] + ['[la] "+v"(t.la)', '[lc] "+v"(t.lc)'] + \
        [f'[w{j}] "=&v"(w[{j}])' for j in range(4)] + [f'[e{j}] "=&v"(e[{j}])' for j in range(2)] + \
        [f'[u{j}] "=&s"(u[{j}])' for j in range(2)] + ['[sk] "=&s"(sk)', '[sv] "=&s"(sv)'] + \
        [f'[{v}] "+s"(t.{v})' for v in ("count", "sb", "ld", "ko", "vo")]
    dma = ['[x] "v"(x)', '[tb] "s"(tb)', '[kb0] "s"(kb0)', '[kb1] "s"(kb1)', '[vb0] "s"(vb0)', '[vb1] "s"(vb1)', '[wp] "s"(wp)',
           '[ring] "s"(ring)', '[end] "s"(end)', '[kind] "s"(kind)', '[bit] "s"(bit)', '[go] "s"(go)']
    out.append("// What quad_steady works on: steps to do; LDS addresses of the first batch and of the wave's part of the batch before it; places of\n"
               "// the group's K and V half tiles in a batch; tiles requested last and lane addresses in the step list (see gen_mfma_pipes.py).\n"
               "struct QuadSteady {\n  int count;\n  uint32_t sb, ld, ko, vo;\n  uint32_t xk[4], xv[4], la, lc;\n};\n\n")
    emit("// t.count times the steps of a run of some kind (quad_steady in gen_mfma_pipes.py), with their barriers; every half step requests the wave's part of the batch that takes the slots of\n"
         "// the batch before it.  ring, end: LDS addresses of the first and past the last batch; wp: the wave's part of a half slot; x, tb: byte offset\n"
         "// of the lane in it, bytes of a tile; kb0, kb1, vb0, vb1: K and V and the same 32 rows further down; bit: of the group in a list entry; go: place of the\n"
         "// group's half tile among four.\n",
         f"quad_steady(int kind, uint32_t ring, uint32_t end, uint32_t wp, uint32_t bit, uint32_t go, {qargs}, const uint32_t (&vl)[4],\n"
         f"                             {oargs}, const void* kb0, const void* kb1, const void* vb0, const void* vb1,\n"
         f"                             uint32_t x, uint32_t tb, QuadSteady& t)",
         "  uint32_t w[4], e[2], u[2], sk, sv;\n", quad_all_steady(), o_ops(nt) + ml + all_state + tiles, kin + vin + cin + dma)
    return "".join(out)


# ---- approximation of the unselected blocks in the quad kernel: a chunk of 32 key blocks per step ----
# On their own the parts of a chunk leave the matrix cores idle during its softmax, and with one workgroup on a compute unit nobody else
# uses them.  So a step takes O += VS^T a and the first-order term of chunk c, and the logits and the weights a of chunk c + 1 in the
# shadow of the 32 MFMAs of the first-order term:
#   O += VS(c)^T a(c);  Z = Kbar(c + 1) Q^T;  W = (scale Hg)^T Q^T, 32 rows at a time, O += A W;  softmax of Z -> a(c + 1), A(c + 1)
# kind 0: that; 1: the group goes on beyond chunk c (no first-order term yet: the weights add up); 2: no next chunk.
# Registers: Z v[152:167], W v[168:199] (two of the four 32-row parts at a time), mask temporaries v[208:211], the rest as elsewhere.  The
# factor for the accumulators where chunk c + 1 raises the maximum (corr) is applied at the beginning of the next step.
FS_Z, FS_U = 152, 208


def approx_weights():
    """items for the logits v[Z:Z+15]: weights and their sums (see stats_step for the mask): P^T -> P0, l += b sum, T6 = sum over both lanes"""
    z, u = (lambda i: vr(FS_Z + i)), (lambda i: vr(FS_U + i % 4))
    t1, t4, t5, t6, t7 = (vr(FS_T + i) for i in (1, 4, 5, 6, 7))
    out = [f"v_lshrrev_b32 {t5}, %[sh], %[unsel]"]
    for i in range(21):  # software pipeline over the 16 elements
        if i < 16:
            out += [f"v_fma_f32 {z(i)}, {z(i)}, %[c], -%[m]", f"v_bfe_i32 {u(i)}, {t5}, {8 * (i // 4) + i % 4}, 1"]
        if 1 <= i <= 16:
            out.append(f"v_exp_f32 {z(i - 1)}, {z(i - 1)}")
        e = i - 3
        if 0 <= e < 16:
            out.append(f"v_and_b32 {z(e)}, {z(e)}, {u(e)}")
        e = i - 4
        if 0 <= e < 16:
            if e == 1:
                out.append(f"v_add_f32 {t4}, {z(0)}, {z(1)}")
            elif e == 3:
                out.append(f"v_add_f32 {t7}, {z(2)}, {z(3)}")
            elif e > 3:
                out.append(f"v_add_f32 {t4 if e % 2 == 0 else t7}, {t4 if e % 2 == 0 else t7}, {z(e)}")
            if e % 2 == 1:
                out.append(f"v_cvt_pk_bf16_f32 {vr(FS_P0 + e // 2)}, {z(e - 1)}, {z(e)}")
    return out + [f"v_add_f32 {t4}, {t4}, {t7}", "s_nop 0", f"v_fmac_f32 %[l], %[bf], {t4}", f"v_mov_b32 {t1}, {t4}",
                  ("s_nop 1", f"v_permlane32_swap_b32 {t4}, {t1}", "s_nop 0"), f"v_add_f32 {t6}, {t4}, {t1}"]


def approx_run(mf, after, prologue):
    """MFMA k of `mf` with its operand fetch issued six MFMAs ahead; load: (tile operand, step, offset) of a row fragment or
    ("v", 16-row step, column tile); the lane addresses of a tile are made when its first fragment is fetched"""
    lines, issued, nbuf, tile = [], [], 6, [None]

    def issue(k):
        f = k % nbuf
        kind, a, b = mf[k]["load"]
        if kind != tile[0]:
            tile[0] = kind
            if kind == "v":
                for t in range(1, 4):
                    lines.append(f"v_xor_b32 {vr(FS_A + 2 * t - 2)}, {hex(t << 6)}, %[av0]")
                    lines.append(f"v_xor_b32 {vr(FS_A + 2 * t - 1)}, {hex(t << 6)}, %[av1]")
            else:
                lines.extend(f"v_xor_b32 {vr(FS_A + st - 1)}, {hex(st << 5)}, %[{kind}]" for st in range(1, 8))
        if kind == "v":
            a0, a1 = ("%[av0]", "%[av1]") if b == 0 else (vr(FS_A + 2 * b - 2), vr(FS_A + 2 * b - 1))
            lines.append(f"ds_read_b64_tr_b16 {Flo(f)}, {a0}{off(a * 32 * QUAD_D)}")
            lines.append(f"ds_read_b64_tr_b16 {Fhi(f)}, {a1}{off(a * 32 * QUAD_D)}")
            issued.append(2)
        else:
            lines.append(f"ds_read_b128 {F(f)}, {f'%[{kind}]' if a == 0 else vr(FS_A + a - 1)}{off(b)}")
            issued.append(1)

    n = len(mf)
    for k in range(min(nbuf, n)):
        issue(k)
    lines += list(prologue)
    for k in range(n):
        outstanding = sum(issued[k + 1:])
        assert outstanding <= 15
        m = mf[k]
        lines += [f"s_waitcnt lgkmcnt({outstanding})", f"{MFMA} {m['acc']}, {F(k % nbuf)}, {m['b']}, {'0' if m['first'] else m['acc']}"]
        if k + nbuf < n:
            issue(k + nbuf)
        lines += after.get(k, [])
    return lines


def approx_body(kind, cold):
    """kind: "both", "more" (no first-order term yet), "last" (no next chunk), "start" (nothing but the first chunk's weights)"""
    D = QUAD_D
    pv = [dict(acc=vr(FS_O + 16 * t, 16), first=False, b=vr(FS_P0 + 4 * ks, 4), load=("v", 2 + ks, t)) for ks in range(2) for t in range(4)]
    qk = [dict(acc=vr(FS_Z, 16), first=(st == 0), b=f"%[q{st}]", load=("ak", st, 0)) for st in range(8)]
    hg = [dict(acc=vr(FS_S0 if k % 2 == 0 else FS_S1, 16), first=(st == 0), b=f"%[q{st}]", load=(f"ah{k // 2}", st, (k % 2) * 64 * D))
          for k in range(4) for st in range(8)]
    corr = "%[corr]"
    pend = [] if kind == "start" else list(pending(cold, None, corr, 64, NOP_AFTER)) + ["s_nop 1"]
    update = lambda k: [f"v_fmac_f32 {vr(FS_O + 16 * k + r)}, %[A], {vr((FS_S0 if k % 2 == 0 else FS_S1) + r)}" for r in range(16)]
    mf = {"both": pv + qk + hg, "more": pv + qk, "last": pv + hg, "start": qk}[kind]
    n, after, tail = len(mf), {}, []
    if kind in ("both", "last"):
        h0 = n - 32
        for k in range(3):
            spread(after, h0 + 8 * (k + 1) + 1, h0 + 8 * (k + 2) - 1, update(k))
        tail += [NOP_AFTER] + update(3)
    if kind != "last":
        grow = growth(cold, None, corr, also=["%[A]"] if kind == "more" else [])
        z0 = n if kind in ("more", "start") else 18  # Z is complete
        items = max_stream(FS_Z) + [grow] + approx_weights()
        if kind == "both":
            pour(after, n, items, first=z0, begin=z0 / n, end=(n - 1) / n)
        else:
            tail += [NOP_AFTER] + flat(items)
        tail.append(f"v_add_f32 %[A], %[A], {vr(FS_T + 6)}" if kind == "more" else f"v_mov_b32 %[A], {vr(FS_T + 6)}")
    return approx_run(mf, after, pend) + tail


def approx_functions():
    D = QUAD_D
    ns, nt = D // 16, D // 32
    clob = ", ".join([f'"v{r}"' for r in list(range(FS_Z, FS_P0)) + list(range(FS_P1, 256))] + ['"memory"', '"scc"', '"vcc"', '"m0"'])
    pa = lambda mode: [f'"{mode}{{v[{200 + 4 * k}:{203 + 4 * k}]}}"(p[{k}])' for k in range(2)]
    out = []
    cold = Cold("as")
    lines = approx_body("start", cold) + [NOP_AFTER] + cold.text()
    text = lambda ls: "\n".join(f'      "{l}\\n\\t"' for l in ls)
    common = q_inputs(D) + ['[c] "s"(c)', '[unsel] "s"(unsel)', '[sh] "v"(sh)', '[bf] "s"(bf)']
    def emit(comment, head, ls, outs, ins):
        out.append(f"{comment}PASA_DEVICE void {head} {{\n  asm volatile(\n{text(ls)}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n      : {clob});\n}}\n\n")
    emit("// Weights of the first chunk of 32 existing, full key blocks (statistics tile + row-fragment offset ak): P^T fragments p, their sum A, and the\n"
         "// factor corr that the accumulators still have to be multiplied by.  unsel, sh, bf: see stats_step.\n",
         f"approx_start(uint32_t ak, const bf16x8 (&q)[{ns}], bf16x8 (&p)[2], float& m, float& l, float& corr, float& A, float c,\n"
         "                              uint32_t unsel, uint32_t sh, float bf)", lines,
         pa("=&") + ['[m] "+v"(m)', '[l] "+v"(l)', '[corr] "=&v"(corr)', '[A] "=&v"(A)'], ['[ak] "v"(ak)'] + common)
    cold = Cold("ap")
    lines = ["s_cmp_eq_u32 %[kind], 0", "s_cbranch_scc0 .Lapother_%="] + approx_body("both", cold) + [".Lapdone_%=:"]
    far = [".Lapother_%=:", "s_cmp_eq_u32 %[kind], 1", "s_cbranch_scc0 .Laplast_%="] + approx_body("more", cold) + ["s_branch .Lapdone_%=", ".Laplast_%=:"] + \
        approx_body("last", cold) + [NOP_AFTER, "s_branch .Lapdone_%="]
    lines += [".subsection 1"] + far + cold.lines + [".subsection 0"]
    emit("// Step of the approximation (kind 0, 1, 2: see gen_mfma_pipes.py).  ak: statistics tile of the next chunk; av0, av1: of this chunk + column-fragment\n"
         "// offsets; ah0, ah1: the two halves of the group's matrix; A: weight of the group so far, on return that of the next chunk's.\n",
         f"approx_step(int kind, uint32_t ak, uint32_t av0, uint32_t av1, uint32_t ah0, uint32_t ah1, const bf16x8 (&q)[{ns}], f32x16 (&o)[{nt}],\n"
         "                             bf16x8 (&p)[2], float& m, float& l, float& corr, float& A, float c, uint32_t unsel, uint32_t sh, float bf)", lines,
         o_ops(nt) + pa("+") + ['[m] "+v"(m)', '[l] "+v"(l)', '[corr] "+v"(corr)', '[A] "+v"(A)'],
         ['[kind] "s"(kind)', '[ak] "v"(ak)', '[av0] "v"(av0)', '[av1] "v"(av1)', '[ah0] "v"(ah0)', '[ah1] "v"(ah1)'] + common)
    return "".join(out)


def run_pipe(D, mf, before, after, dmas, waves):
    """MFMA k of `mf` with its operand fetch issued six MFMAs ahead; `before[k]` / `after[k]` are instruction
    lists placed right before / after MFMA k; `dmas`: tile-load instructions (slot tag, index), one per MFMA
    shadow from the first MFMA on."""
    lines = []
    pipe = LdsPipe(lines, D)
    pipe.k_addresses()
    n = len(mf)
    for k in range(min(pipe.nbuf, n)):
        pipe.issue(k, mf[k]["load"])
    dmas = list(dmas)
    for k in range(n):
        pipe.wait_for(k)
        lines += before.get(k, [])
        m = mf[k]
        lines.append(f"{MFMA} {m['acc']}, {F(k % pipe.nbuf)}, {m['b']}, {'0' if m['first'] else m['acc']}")
        if dmas:
            lines.append(f"s_add_u32 m0, %[l{dmas[0][0]}], {hex(dmas[0][1] * waves * 1024)}")
        if k + pipe.nbuf < n:
            pipe.issue(k + pipe.nbuf, mf[k + pipe.nbuf]["load"])
        elif dmas:
            lines.append("s_nop 0")
        if dmas:
            which, jj = dmas.pop(0)
            lines.append(f"global_load_lds_dwordx4 %[x{jj}], %[{which}b]")
        lines += after.get(k, [])
    assert not dmas
    return lines


def flat(stream):
    out = []
    for item in stream:
        out += list(item) if isinstance(item, tuple) else [item]
    return out


# ---- zeroth-order step of the approximation: one chunk of 32 key blocks, all of them existing and of full size ----
#   Z = Kbar Q^T  (rows 0..31 of the statistics tile; the next tile of the stream is requested in the shadow)
#   a_j = exp2(c z_j - m) for the unselected blocks, 0 for the selected ones; l += b sum a_j; A = sum a_j
#   O += VS^T a   (rows 32..63), the first half of it while the second half of the a_j is still being computed
# A selected block takes part in the running maximum, which is taken over the unmasked logits: its mean-key logit
# exceeds the largest logit of its keys, which this workgroup's exact passes have seen, by the rounding of the mean
# at most, so the maximum stays that of terms that are summed.  (Were the maximum masked, a selected block's a_j
# could overflow before its mask is applied.)  Lane (x, h) holds block 8g + 4h + r
# in register 4g + r, so with the bitmap word shifted right by 4h the block's bit is bit 8g + r for every lane.
# Registers: Z v[168:183], per-element masks v[184:199], P^T v[200:207], the rest as in fused_step.
def stats_step(D, waves):
    ns, nt = D // 16, D // 32
    ni = tile_loads(D, waves)
    n_o = 16 * nt
    S, U, P = FS_S0, FS_S1, FS_P0
    s = lambda i: vr(S + i)
    u = lambda i: vr(U + i)
    t4, t5, t7 = vr(FS_T + 4), vr(FS_T + 5), vr(FS_T + 7)
    mf = [dict(acc=vr(S, 16), first=(st == 0), b=f"%[q{st}]", load=("k", st, 0)) for st in range(ns)]
    for ks2 in range(2):
        for t in range(nt):
            mf.append(dict(acc=vr(FS_O + 16 * t, 16), first=False, b=vr(P + 4 * ks2, 4), load=("v", 2 + ks2, t)))
    pre = [f"v_lshrrev_b32 {t5}, %[sh], %[unsel]"] + max_stream(S) + raise_max(n_o, True)
    first_half, second_half = [], []
    for i in range(21):  # software pipeline over the 16 elements
        cur = first_half if i - 4 < 8 and i < 12 else second_half
        if i < 16:
            cur.append(f"v_fma_f32 {s(i)}, {s(i)}, %[c], -%[m]")
            cur.append(f"v_bfe_i32 {u(i)}, {t5}, {8 * (i // 4) + i % 4}, 1")
        if 1 <= i <= 16:
            cur.append(f"v_exp_f32 {s(i - 1)}, {s(i - 1)}")
        e = i - 3
        if 0 <= e < 16:
            cur.append(f"v_and_b32 {s(e)}, {s(e)}, {u(e)}")
        e = i - 4
        if 0 <= e < 16:
            if e == 1:
                cur.append(f"v_add_f32 {t4}, {s(0)}, {s(1)}")
            elif e == 3:
                cur.append(f"v_add_f32 {t7}, {s(2)}, {s(3)}")
            elif e > 3:
                cur.append(f"v_add_f32 {t4 if e % 2 == 0 else t7}, {t4 if e % 2 == 0 else t7}, {s(e)}")
            if e % 2 == 1:
                cur.append(f"v_cvt_pk_bf16_f32 {vr(P + e // 2)}, {s(e - 1)}, {s(e)}")
    t1 = vr(FS_T + 1)
    fin = [f"v_add_f32 {t4}, {t4}, {t7}", "s_nop 0", f"v_fmac_f32 %[l], %[bf], {t4}", f"v_mov_b32 {t1}, {t4}", "s_nop 1",
           f"v_permlane32_swap_b32 {t4}, {t1}", "s_nop 0", f"v_add_f32 %[A], {t4}, {t1}"]
    before = {ns: [NOP_AFTER] + flat(pre) + first_half + ["s_nop 1"], ns + nt: ["s_nop 1"]}
    after = {}
    spread(after, ns, ns + nt - 1, second_half)
    spread(after, ns + nt, ns + 2 * nt - 1, fin)
    lines = run_pipe(D, mf, before, after, [("s", j) for j in range(ni)], waves)
    lines.append(NOP_AFTER)
    return lines


# ---- first-order step: 64 value columns of one group,  O^T[part] += A ((scale Hg)^T[part] Q^T) ----
# Rows 0..31 of the tile first, then rows 32..63 with the update from the first product in the shadow of
# their MFMAs.  The next tile of the stream is requested in the shadow of the first MFMAs.
def first_order_step(D, part, waves):
    ns = D // 16
    ni = tile_loads(D, waves)
    mf = []
    for half in range(2):
        for st in range(ns):
            mf.append(dict(acc=vr(FS_S0 if half == 0 else FS_S1, 16), first=(st == 0), b=f"%[q{st}]", load=("k", st, half)))
    o0, o1 = FS_O + 32 * part, FS_O + 32 * part + 16
    after = {}
    spread(after, ns + 1, 2 * ns - 1, [f"v_fmac_f32 {vr(o0 + r)}, %[A], {vr(FS_S0 + r)}" for r in range(16)])
    lines = run_pipe(D, mf, {}, after, [("s", j) for j in range(ni)], waves)
    lines.append(NOP_AFTER)
    lines += [f"v_fmac_f32 {vr(o1 + r)}, %[A], {vr(FS_S1 + r)}" for r in range(16)]
    return lines


def asm_block(lines, outs, ins, extra_clobbers=()):
    text = "\n".join(f'      "{l}\\n\\t"' for l in lines)
    clob = ", ".join([f'"v{r}"' for r in range(CLOBBER_LO, CLOBBER_HI + 1)] + [f'"{c}"' for c in extra_clobbers])
    return f"  asm volatile(\n{text}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n      : {clob});\n"


def logits_softmax(D):
    """The first half of fused_step for loops that must meet a barrier before P V (the V tile lands later):
    S0, S1 = K Q^T with the softmax of S0 in the shadow of the MFMAs of S1, then the softmax of S1; leaves
    P0, P1.  No MFMA adds to the accumulators meanwhile, so both halves rescale them at once; the weights of the
    first half stay fp32 until the second half has settled the maximum."""
    ns, nt = D // 16, D // 32
    ni = (64 // (1024 // (2 * D))) // 4
    n_o = 16 * nt
    mf = []
    for half in range(2):
        for st in range(ns):
            mf.append(dict(acc=vr(FS_S0 if half == 0 else FS_S1, 16), first=(st == 0), b=f"%[q{st}]", load=("k", st, half)))
    n = len(mf)
    after = {}
    spread(after, ns + 1, n - 1, max_stream(FS_S0) + raise_max(n_o, True) + exp_stream(FS_S0, FS_P0, convert=False))
    lines = []
    pipe = LdsPipe(lines, D)
    pipe.k_addresses()
    for k in range(pipe.nbuf):
        pipe.issue(k, mf[k]["load"])
    dmas = [("k", j) for j in range(ni)] + [("v", j) for j in range(ni)]
    for k in range(n):
        pipe.wait_for(k)
        m = mf[k]
        lines.append(f"{MFMA} {m['acc']}, {F(k % pipe.nbuf)}, {m['b']}, {'0' if m['first'] else m['acc']}")
        if dmas:
            lines.append(f"s_add_u32 m0, %[l{dmas[0][0]}], {hex(dmas[0][1] * 4096)}")
        if k + pipe.nbuf < n:
            pipe.issue(k + pipe.nbuf, mf[k + pipe.nbuf]["load"])
        elif dmas:
            lines.append("s_nop 0")
        if dmas:
            which, jj = dmas.pop(0)
            lines.append(f"global_load_lds_dwordx4 %[x{jj}], %[{which}b]")
        lines += after.get(k, [])
    assert not dmas
    lines.append(NOP_AFTER)  # the last MFMA of S1 has to deliver before its maximum is taken
    # the weights of the first half are still fp32: if the second half raises the maximum they follow it
    for item in max_stream(FS_S1) + raise_max(n_o, True, also=[vr(FS_S0 + i) for i in range(16)]) + \
            convert_stream(FS_S0, FS_P0) + exp_stream(FS_S1, FS_P1):
        lines += list(item) if isinstance(item, tuple) else [item]
    # raise_max(.., True) is used twice in this sequence: make its labels distinct
    seen, out = 0, []
    for l in lines:
        if "Lfs_keepa" in l:
            l = l.replace("Lfs_keepa", "Lfs_keepa" if seen < 2 else "Lfs_keepc")
            seen += 1
        out.append(l)
    return out


# Operands that are MFMA results or inputs of several sequences are bound to the same registers everywhere,
# which leaves the register allocator nothing to get wrong: accumulators O v[0:63], logits v[168:199],
# P^T fragments v[200:215].
def o_ops(nt):
    return [f'[o{t}] "+{{v[{FS_O + 16 * t}:{FS_O + 16 * t + 15}]}}"(o[{t}])' for t in range(nt)]


def c_ops():
    return ['[c0] "=&{v[168:183]}"(c0)', '[c1] "=&{v[184:199]}"(c1)']


def p_ops(nks):
    return [f'[p{k}] "{{v[{200 + 4 * k}:{200 + 4 * k + 3}]}}"(p[{k}])' for k in range(nks)]


def q_inputs(D):
    return [f'[q{s}] "v"(q[{s}])' for s in range(D // 16)]


def gen():
    out = []
    out.append("// GENERATED by gen_mfma_pipes.py -- do not edit.  Software-pipelined LDS-read + MFMA sequences of the\n"
               "// attention kernel (gfx950).  Every function is one asm statement; v226..v255 are its operand buffers.\n"
               "#pragma once\n#include \"pasa_device.hpp\"\n\nnamespace pipes {\n\n"
               "// What one pipelined step hands to the next: the logits of the second half of the tile whose P V comes next, the weights of\n"
               "// its first half, and the factor for the accumulators (where flag is not zero).\n"
               "struct PipeState {\n  f32x16 s1;\n  bf16x8 p0[2];\n  float corr;\n  uint64_t flag;\n};\n\n")
    for D in (128, 64):
        ni = (64 // (1024 // (2 * D))) // 4
        # rows_x_q
        out.append(f"// c0 = (tile rows 0..31) x Q^T, c1 = (tile rows 32..63) x Q^T;  a = tile address + lane's row-fragment offset\n"
                   f"PASA_DEVICE void rows_x_q(uint32_t a, const bf16x8 (&q)[{D // 16}], f32x16& c0, f32x16& c1) {{\n")
        out.append(asm_block(rows_x_q(D, True, 0), c_ops(), ['[a] "v"(a)'] + q_inputs(D), ("memory",)))
        out.append("}\n\n")
        for waves in (4, 8):
            ni = tile_loads(D, waves)
            out.append(f"// the same, and in the shadow of the first MFMAs this wave's share of the next K tile (from kb into the slot\n"
                       f"// at LDS address lk) and V tile (vb, lv) is requested; x = the lane's byte offsets of its {ni} loads per tile\n"
                       f"// ({waves} waves)\n"
                       f"PASA_DEVICE void rows_x_q_dma(uint32_t a, const bf16x8 (&q)[{D // 16}], f32x16& c0, f32x16& c1, const void* kb,\n"
                       f"                             const void* vb, const uint32_t (&x)[{ni}], uint32_t lk, uint32_t lv) {{\n")
            ins = ['[a] "v"(a)'] + q_inputs(D) + ['[kb] "s"(kb)', '[vb] "s"(vb)', '[lk] "s"(lk)', '[lv] "s"(lv)'] + \
                  [f'[x{j}] "v"(x[{j}])' for j in range(ni)]
            out.append(asm_block(rows_x_q(D, True, ni, waves), c_ops(), ins, ("memory", "scc", "m0")))
            out.append("}\n\n")
        ni = tile_loads(D, 4)
        out.append(f"// rows 0..31 only: c0 + c1 = (tile rows 0..31) x Q^T (even contraction steps in c0, odd ones in c1)\n"
                   f"PASA_DEVICE void rows32_x_q(uint32_t a, const bf16x8 (&q)[{D // 16}], f32x16& c0, f32x16& c1) {{\n")
        out.append(asm_block(rows_x_q(D, False, 0), c_ops(), ['[a] "v"(a)'] + q_inputs(D), ("memory",)))
        out.append("}\n\n")
        for name, nks, row0 in (("cols_x_p64", 4, 0), ("cols_x_p32_hi", 2, 32)):
            nt = D // 32
            out.append(f"// o[t] += (tile rows {row0}..{row0 + 16 * nks - 1}, value columns 32t..32t+31)^T x p;  a0, a1 = tile address + the lane's\n"
                       f"// column-fragment offsets (rows 0.. and rows 8..)\n"
                       f"PASA_DEVICE void {name}(uint32_t a0, uint32_t a1, const bf16x8 (&p)[{nks}], f32x16 (&o)[{nt}]) {{\n")
            outs = o_ops(nt)
            ins = ['[a0] "v"(a0)', '[a1] "v"(a1)'] + p_ops(nks)
            out.append(asm_block(cols_x_p(D, nks, row0), outs, ins, ("memory",)))
            out.append("}\n\n")
        nt = D // 32
        out.append(f"// cols_x_p64, and in the shadow of the first MFMAs this wave's share of two more tiles is requested (see rows_x_q_dma)\n"
                   f"PASA_DEVICE void cols_x_p64_dma(uint32_t a0, uint32_t a1, const bf16x8 (&p)[4], f32x16 (&o)[{nt}], const void* kb,\n"
                   f"                               const void* vb, const uint32_t (&x)[{ni}], uint32_t lk, uint32_t lv) {{\n")
        outs = o_ops(nt)
        ins = ['[a0] "v"(a0)', '[a1] "v"(a1)'] + p_ops(4) + \
              ['[kb] "s"(kb)', '[vb] "s"(vb)', '[lk] "s"(lk)', '[lv] "s"(lv)'] + [f'[x{j}] "v"(x[{j}])' for j in range(ni)]
        out.append(asm_block(cols_x_p(D, 4, 0, ni), outs, ins, ("memory", "scc", "m0")))
        out.append("}\n\n")
    out.append(pipe_functions())
    out.append(quad_functions())
    out.append(approx_functions())
    for D, waves in ((128, 4), (128, 2), (64, 4), (64, 2)):
        ns, nt = D // 16, D // 32
        ni = tile_loads(D, waves)
        out.append(f"// One whole 64-key tile (all keys valid) against the wave's 32 queries: logits, online softmax, P V.\n"
                   f"// ak, av0, av1: K tile address + row-fragment offset, V tile address + the two column-fragment offsets;\n"
                   f"// m, l: running maximum (log2 units) and normaliser share; c = scale * log2(e); kb/vb/x/lk/lv: the next pair\n"
                   f"// of tiles to request (see rows_x_q_dma), by {waves} waves.\n"
                   f"PASA_DEVICE void fused_step(uint32_t ak, uint32_t av0, uint32_t av1, const bf16x8 (&q)[{ns}], f32x16 (&o)[{nt}],\n"
                   f"                           float& m, float& l, float c, const void* kb, const void* vb,\n"
                   f"                           const uint32_t (&x)[{ni}], uint32_t lk, uint32_t lv) {{\n"
                   f"  uint64_t flag;\n")
        outs = o_ops(nt) + \
               ['[m] "+v"(m)', '[l] "+v"(l)', '[flag] "=&s"(flag)']
        ins = ['[ak] "v"(ak)', '[av0] "v"(av0)', '[av1] "v"(av1)', '[c] "s"(c)'] + q_inputs(D) + \
              ['[kb] "s"(kb)', '[vb] "s"(vb)', '[lk] "s"(lk)', '[lv] "s"(lv)'] + [f'[x{j}] "v"(x[{j}])' for j in range(ni)]
        text = "\n".join(f'      "{l}\\n\\t"' for l in fused_step(D, waves))
        clob = ", ".join([f'"v{r}"' for r in range(FUSED_CLOBBER_LO, 256)] + ['"memory"', '"scc"', '"vcc"', '"m0"'])
        out.append(f"  asm volatile(\n{text}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n      : {clob});\n}}\n\n")
    for D in (128, 64):
        ns, nt = D // 16, D // 32
        ni = (64 // (1024 // (2 * D))) // 4
        out.append(f"// Logits and online softmax of one whole 64-key tile (all keys valid); leaves the P^T fragments p.  Two more\n"
                   f"// tiles are requested meanwhile (see rows_x_q_dma).  Arguments as in fused_step.\n"
                   f"PASA_DEVICE void logits_softmax(uint32_t ak, const bf16x8 (&q)[{ns}], f32x16 (&o)[{nt}], float& m, float& l, float c,\n"
                   f"                               bf16x8 (&p)[4], const void* kb, const void* vb, const uint32_t (&x)[{ni}],\n"
                   f"                               uint32_t lk, uint32_t lv) {{\n")
        outs = o_ops(nt) + ['[m] "+v"(m)', '[l] "+v"(l)'] + \
               [f'[p{k}] "=&{{v[{200 + 4 * k}:{200 + 4 * k + 3}]}}"(p[{k}])' for k in range(4)]
        ins = ['[ak] "v"(ak)', '[c] "s"(c)'] + q_inputs(D) + \
              ['[kb] "s"(kb)', '[vb] "s"(vb)', '[lk] "s"(lk)', '[lv] "s"(lv)'] + [f'[x{j}] "v"(x[{j}])' for j in range(ni)]
        text = "\n".join(f'      "{l}\\n\\t"' for l in logits_softmax(D))
        clob = ", ".join([f'"v{r}"' for r in range(168, 200)] + [f'"v{r}"' for r in range(216, 256)] +
                         ['"memory"', '"scc"', '"vcc"', '"m0"'])
        out.append(f"  asm volatile(\n{text}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n      : {clob});\n}}\n\n")
    for D, waves in ((128, 4), (64, 4)):
        ns, nt = D // 16, D // 32
        ni = tile_loads(D, waves)
        dma_ins = ['[sb] "s"(sb)', '[ls] "s"(ls)'] + [f'[x{j}] "v"(x[{j}])' for j in range(ni)]
        out.append(f"// Zeroth-order step of the approximation for a chunk of 32 existing, full key blocks.  ak, av0, av1: the\n"
                   f"// statistics tile's address + row-fragment / column-fragment offsets; unsel: bit x set iff block x of the\n"
                   f"// chunk is NOT selected; sh = 4 * (lane >> 5); bf = tokens per block; A <- sum of the chunk's weights a_j.\n"
                   f"// One more tile (from sb into the slot at LDS address ls) is requested meanwhile ({waves} waves).\n"
                   f"PASA_DEVICE void stats_step(uint32_t ak, uint32_t av0, uint32_t av1, const bf16x8 (&q)[{ns}], f32x16 (&o)[{nt}],\n"
                   f"                           float& m, float& l, float c, uint32_t unsel, uint32_t sh, float bf, float& A,\n"
                   f"                           const void* sb, const uint32_t (&x)[{ni}], uint32_t ls) {{\n")
        outs = o_ops(nt) + ['[m] "+v"(m)', '[l] "+v"(l)', '[A] "=&v"(A)']
        ins = ['[ak] "v"(ak)', '[av0] "v"(av0)', '[av1] "v"(av1)', '[c] "s"(c)', '[unsel] "s"(unsel)', '[sh] "v"(sh)',
               '[bf] "s"(bf)'] + q_inputs(D) + dma_ins
        text = "\n".join(f'      "{l}\\n\\t"' for l in stats_step(D, waves))
        clob = ", ".join([f'"v{r}"' for r in range(FUSED_CLOBBER_LO, 256)] + ['"memory"', '"scc"', '"vcc"', '"m0"'])
        out.append(f"  asm volatile(\n{text}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n      : {clob});\n}}\n\n")
        for part in range(D // 64):
            out.append(f"// First-order step: o[{2 * part}], o[{2 * part + 1}] += A * (tile x Q^T), the tile being rows {64 * part}..{64 * part + 63} of the\n"
                       f"// group's (scale Hg)^T; a = tile address + row-fragment offset; one more tile is requested (see stats_step).\n"
                       f"PASA_DEVICE void first_order_step{part}(uint32_t ak, const bf16x8 (&q)[{ns}], f32x16 (&o)[{nt}], float A,\n"
                       f"                                 const void* sb, const uint32_t (&x)[{ni}], uint32_t ls) {{\n")
            outs = [o_ops(nt)[2 * part], o_ops(nt)[2 * part + 1]]
            ins = ['[ak] "v"(ak)', '[A] "v"(A)'] + q_inputs(D) + dma_ins
            text = "\n".join(f'      "{l}\\n\\t"' for l in first_order_step(D, part, waves))
            out.append(f"  asm volatile(\n{text}\n      : {', '.join(outs)}\n      : {', '.join(ins)}\n      : {clob});\n}}\n\n")
    out.append("}  // namespace pipes\n")
    return "".join(out)


if __name__ == "__main__":
    here = os.path.dirname(os.path.abspath(__file__))
    with open(os.path.join(here, "pasa_mfma_pipes.hpp"), "w") as f:
        f.write(gen())
