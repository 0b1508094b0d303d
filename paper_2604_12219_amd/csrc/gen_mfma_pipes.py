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


def fused_step(D):
    ns, nt = D // 16, D // 32
    ni = (64 // (1024 // (2 * D))) // 4
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


def growth(cold, flag, corr):
    """after max_stream: where the maximum grew for some lane, m, l and the factor `corr` for the accumulators; `flag` is not
    zero then.  (The lane's own maximum decides, see raise_max.)"""
    t0, t1, t2 = (vr(FS_T + i) for i in range(3))
    body = [f"v_mov_b32 {t1}, {t0}", "s_nop 1", f"v_permlane32_swap_b32 {t0}, {t1}", "s_nop 0",
            f"v_max3_f32 {t1}, %[m], {t0}, {t1}", f"v_sub_f32 {t2}, %[m], {t1}", f"v_exp_f32 {corr}, {t2}",
            f"v_mov_b32 %[m], {t1}", "s_nop 0", f"v_mul_f32 %[l], %[l], {corr}"]
    return tuple([f"v_cmp_gt_f32 vcc, {t0}, %[m]", f"s_mov_b64 {flag}, vcc"] + cold.block("s_cbranch_vccnz", body))


def pending(cold, flag, corr, n_o, nop):
    """accumulators *= corr if flag is not zero"""
    return tuple([f"s_cmp_lg_u64 {flag}, 0"] +
                 cold.block("s_cbranch_scc1", [nop] + [f"v_mul_f32 {vr(FS_O + i)}, {vr(FS_O + i)}, {corr}" for i in range(n_o)]))


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
    for D in (128, 64):
        ns, nt = D // 16, D // 32
        ni = (64 // (1024 // (2 * D))) // 4
        out.append(f"// One whole 64-key tile (all keys valid) against the wave's 32 queries: logits, online softmax, P V.\n"
                   f"// ak, av0, av1: K tile address + row-fragment offset, V tile address + the two column-fragment offsets;\n"
                   f"// m, l: running maximum (log2 units) and normaliser share; c = scale * log2(e); kb/vb/x/lk/lv: the next pair\n"
                   f"// of tiles to request (see rows_x_q_dma).\n"
                   f"PASA_DEVICE void fused_step(uint32_t ak, uint32_t av0, uint32_t av1, const bf16x8 (&q)[{ns}], f32x16 (&o)[{nt}],\n"
                   f"                           float& m, float& l, float c, const void* kb, const void* vb,\n"
                   f"                           const uint32_t (&x)[{ni}], uint32_t lk, uint32_t lv) {{\n"
                   f"  uint64_t flag;\n")
        outs = o_ops(nt) + \
               ['[m] "+v"(m)', '[l] "+v"(l)', '[flag] "=&s"(flag)']
        ins = ['[ak] "v"(ak)', '[av0] "v"(av0)', '[av1] "v"(av1)', '[c] "s"(c)'] + q_inputs(D) + \
              ['[kb] "s"(kb)', '[vb] "s"(vb)', '[lk] "s"(lk)', '[lv] "s"(lv)'] + [f'[x{j}] "v"(x[{j}])' for j in range(ni)]
        text = "\n".join(f'      "{l}\\n\\t"' for l in fused_step(D))
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
                   f"// One more tile (from sb into the slot at LDS address ls) is requested meanwhile.\n"
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
