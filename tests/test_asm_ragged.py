"""The ragged attention stream (gen_attn_fwd128x2.py --ragged) on the CPU: the hazard distances of
test_asm_hazards.py, and the execution model of test_asm_model.py extended by what this stream adds: per-lane
offsets that are clamped at the head's last row, stores under a narrowed execution mask, rounds that
are pairs of blocks.  Checked for whole workgroups: no access outside the tensors, every row that
exists sees the right keys in LDS, every row is written exactly once and no other is."""
import os
import random
import re
import subprocess
import sys

import pytest

import test_asm_hazards
from test_asm_hazards import *  # noqa: F401,F403  (its tests run here on the ragged stream)
from test_asm_model import KBASE, LBASE, M32, OBASE, QBASE, RING, VBASE, Wave, kv_division

GEN = test_asm_hazards.GEN


def generated(tmp_path_factory):
    path = tmp_path_factory.mktemp("gen") / "ragged.inc"
    subprocess.run([sys.executable, GEN, "--ragged", str(path)], check=True, capture_output=True)
    return path.read_text()


@pytest.fixture(scope="module")
def stream(tmp_path_factory):
    text = generated(tmp_path_factory)
    lines = re.findall(r'^\s+"([^"\\]*)\\n" \\$', text, flags=re.M)
    clob = re.search(r"#define A2SF_FWD128X2R_CLOBBERS (.*)", text).group(1)
    return [ln.strip() for ln in lines if ln.strip() and not ln.strip().startswith(";")], clob


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    prog, labels = [], {}
    for ln in re.findall(r'^\s+"([^"\\]*)\\n" \\$', generated(tmp_path_factory), flags=re.M):
        ln = ln.strip()
        if ln.endswith(":"):
            labels[ln[:-1]] = len(prog)
        elif ln.startswith(";"):
            prog.append(("marker", ln))
        elif ln:
            op, _, rest = ln.partition(" ")
            prog.append((op, [a.strip() for a in rest.split(",")] if rest else []))
    return prog, labels


def signed(x):
    return x - (1 << 32) if x & 0x80000000 else x


class RaggedWave(Wave):
    def __init__(self, *a):
        super().__init__(*a)
        self.reg = {}          # per-lane offset registers: (added to the lane's own offset, upper limit)
        self.exec = None       # byte limit of the narrowed execution mask

    def run(self):
        while self.pc < len(self.prog):
            op, a = self.prog[self.pc]
            if op == "v_add_u32" and a[2] in ("%[kl0]", "%[vl0]"):
                self.reg[a[0]] = (int(a[1], 0), 1 << 40)
            elif op == "v_min_u32" and a[2] == "%[qoff]":
                self.reg[a[0]] = (0, self.val(a[1]))
            elif op == "v_min_u32":
                assert a[0] == a[2]
                self.reg[a[0]] = (self.reg[a[0]][0], self.val(a[1]))
            elif op == "v_cmpx_gt_i32":
                assert self.exec is None
                self.exec = (signed(self.val(a[1])), a[2])
            elif op == "s_mov_b64" and a[0] == "exec":
                self.exec = None
            elif self.exec is not None:
                assert op == "s_nop" or op.startswith("global_store"), f"{op} under a narrowed mask"
            # one instruction of the base model
            here, prog = self.pc, self.prog
            self.prog = _Upto(prog, here + 1)
            stopped = super().run()
            self.prog = prog
            if stopped:
                return True
        return False

    def s_min_u32(self, a):
        x, y = self.val(a[1]) & M32, self.val(a[2]) & M32
        self.put(a[0], min(x, y))
        self.scc = int(x < y)

    def s_min_i32(self, a):
        x, y = signed(self.val(a[1]) & M32), signed(self.val(a[2]) & M32)
        self.put(a[0], min(x, y) & M32)
        self.scc = int(x < y)

    def global_load_lds_dwordx4(self, a):
        add, lim = self.reg[a[0]]
        off = self._offset(a)
        slot = (self.s["m0"] + off) & M32
        u = (slot - 1024 * self.wave) % 16384 // 4096
        ptr = self.val(a[1].split()[0])
        lanes = []             # (row in tile, first byte, byte after the last) as addressed
        for rr in range(4):
            lrow = 4 * self.wave + rr
            first, last = min(lrow * 256 + add, lim) + off, min(lrow * 256 + 240 + add, lim) + off
            lanes.append((16 * u + lrow, ptr + first, ptr + last + 16))
        ev = {"wave": self.wave, "issued": self.epoch, "retired": None, "lds": slot, "u": u, "ptr": ptr, "lanes": lanes}
        self.dma.append(ev)
        self.vm.append(ev)

    def global_load_dwordx4(self, a):
        add, lim = self.reg[a[1]]
        self.qloads.append((self.val(a[2].split()[0]) + self._offset(a), lim, self.s[50]))
        self.qevents.append({"retired": None})
        self.vm.append(self.qevents[-1])

    def global_store_dword(self, a):
        lim, reg = self.exec
        assert reg == "%[l32x4]" == a[0]
        self.stores.append(("lse", self.val(a[2].split()[0]), max(0, min(lim, 128)) // 4))
        self.vm.append(None)

    def global_store_dwordx4(self, a):
        lim, reg = self.exec
        assert reg == "%[lanex16]" == a[0]
        self.stores.append(("o", self.val(a[2].split()[0]) + self._offset(a), max(0, min(lim, 1024)) // 256))
        self.vm.append(None)


class _Upto:
    """A program that ends before instruction `end`, for running one instruction at a time; branches
    inside it go where they go."""

    def __init__(self, prog, end):
        self.prog, self.end, self.first = prog, end, True

    def __len__(self):
        return self.end if self.first else 0

    def __getitem__(self, i):
        self.first = False
        return self.prog[i]


def run_workgroup(program, n, G, kvr, first, second, nqb, seed=None, rounds=1, vid0=0):
    prog, labels = program
    rng = random.Random(seed)
    coin = (lambda: rng.random() < 0.15) if seed is not None else (lambda: False)
    waves = []
    for w in range(4):
        operands = dict(qlo=QBASE & M32, qhi=QBASE >> 32, klo=KBASE & M32, khi=KBASE >> 32,
                        vlo=VBASE & M32, vhi=VBASE >> 32, olo=OBASE & M32, ohi=OBASE >> 32,
                        llo=LBASE & M32, lhi=LBASE >> 32, n=n, g0=first[0], qb0=first[1], vid0=vid0, rounds=rounds,
                        nqm=(1 << 32) // nqb + 1, nqbm1=nqb - 1, kvs=kv_division(kvr)[0], kvm=kv_division(kvr)[1],
                        w32a=32 * w, w32b=32 * (7 - w), wodd=w & 1, wave_lds=1024 * w, scale=0,
                        hx16=0, krow=0, clvs16=0, vrow=0, kl0=0, vl0=0, qoff=0, lv=0, l32x4=0,
                        lanex16=0, strip_w=0, x16=0, crr16=0, strip_r=0)
        waves.append(RaggedWave(prog, labels, operands, w, coin))
    live = [True] * 4
    while any(live):
        live = [wv.run() for wv in waves]
        assert all(live) or not any(live), "the waves of a workgroup pass different numbers of barriers"
    return waves


def check_workgroup(waves, blocks, n, G, kvr):
    heads_kv = -(-G // kvr)
    tiles = -(-n // 64)
    rounds = len(blocks)
    assert len({wv.epoch for wv in waves}) == 1
    fills = {}
    for wv in waves:
        for ev in wv.dma:
            kind, base = ("K", KBASE) if ev["ptr"] < VBASE else ("V", VBASE)
            head, inside = divmod(ev["ptr"] - base, n * 256)
            tile, within = divmod(inside, 16384)
            assert within == 0
            stage, slot = divmod(ev["lds"], 32768)
            assert 0 <= ev["lds"] < RING and (slot >= 16384) == (kind == "V")
            assert slot % 16384 == 4096 * ev["u"] + 1024 * wv.wave
            for row, lo, hi in ev["lanes"]:
                assert base <= lo and hi <= base + heads_kv * n * 256, "fetch outside K / V"
                if tile * 64 + row < n:
                    assert lo == ev["ptr"] + row * 256 and hi == lo + 256, "a row that exists was clamped"
            ev.update(head=head, tile=tile)
            fills.setdefault((kind, stage), {}).setdefault(wv.wave, []).append(ev)
    for wv in waves:
        for rd in wv.reads:
            g, qb = blocks[rd["round"]]
            nt, t = 4 * qb + 4, rd["t"]
            if rd["phase"] == "block":
                want = rd["stage"]
                assert rd["kind"] == "K" and want in (0, 1)
            elif rd["phase"] == "X":
                want = t + 1 if rd["kind"] == "K" else t
            elif rd["phase"] == "Y":
                want = t if rd["kind"] == "V" else t + 2
            else:
                want = t
            assert want % 4 == rd["stage"]
            head, tile = (g, want) if want < nt else blocks[min(rd["round"] + 1, rounds - 1)][:1] + (want - nt,)
            for w2 in range(4):
                mine = [ev for ev in fills[(rd["kind"], rd["stage"])][w2] if ev["issued"] <= rd["epoch"]]
                assert len(mine) >= 4
                if want >= nt and rd["round"] + 1 >= rounds:
                    continue
                for last in mine[-4:]:
                    if not tiles <= want < nt:      # (no row that exists reads a tile past the rows)
                        assert (last["head"], last["tile"]) == (head // kvr, tile), (rd, last)
                    assert last["retired"] is not None and last["retired"] < rd["epoch"], (rd, last)
                assert {ev["u"] for ev in mine[-4:]} == {0, 1, 2, 3}
    for wv in waves:
        exp_o, exp_l, q_rows = set(), set(), {}
        for j, (g, qb) in enumerate(blocks):
            for b, f in ((0, 32 * wv.wave), (1, 32 * (7 - wv.wave))):
                rows = {g * n + r for r in range(256 * qb + f, min(256 * qb + f + 32, n))}
                exp_o |= rows
                exp_l |= rows
                q_rows.setdefault(j, []).append((g, 256 * qb + f))
        got_o, got_l = [], []
        for kind, addr, count in wv.stores:
            base, size, out = (OBASE, 256, got_o) if kind == "o" else (LBASE, 4, got_l)
            out += [(addr - base) // size + i for i in range(count)]
        assert sorted(got_o) == sorted(exp_o) and sorted(got_l) == sorted(exp_l)
        loads = {}
        for addr, lim, j in wv.qloads:
            loads.setdefault(j, []).append((addr, lim))
            for l32 in range(32):
                for h in (0, 1):
                    at = addr + min(l32 * 256 + 16 * h, lim)
                    assert QBASE <= at and at + 16 <= QBASE + G * n * 256, "Q outside the tensor"
        # the loads of round j: setup (j = 0) and the last tile of round j - 1, in order
        seq = [x for j in sorted(loads) for x in loads[j]]
        order = [0] + [min(j + 1, rounds - 1) for j in range(rounds)]
        assert len(seq) == 16 * len(order)
        for k, j in enumerate(order):
            for b, (g, row) in enumerate(q_rows[j]):
                for kk in range(8):
                    addr, lim = seq[16 * k + 8 * b + kk]
                    for l32 in range(32):
                        if row + l32 < n:
                            for h in (0, 1):
                                assert addr + min(l32 * 256 + 16 * h, lim) == QBASE + (g * n + row + l32) * 256 + 32 * kk + 16 * h


def pair_blocks(vid0, rounds, nqb):
    out = []
    for j in range(rounds):
        a, p = divmod(vid0 + 32 * (j >> 1), nqb)
        out.append((2 * a + (j & 1), p if j & 1 else nqb - 1 - p))
    return out


@pytest.mark.parametrize("n", [513, 575, 576, 577, 640, 769, 1000, 1023, 1024, 2049, 3001])
def test_single_blocks(program, n):
    """One workgroup per row block: the last block with one row, up to and past a tile's edge, full."""
    nqb = -(-n // 256)
    for G, kvr, g in ((1, 1, 0), (6, 3, 5)):
        for qb in {0, nqb - 2, nqb - 1}:
            waves = run_workgroup(program, n, G, kvr, (g, qb), None, nqb)
            check_workgroup(waves, [(g, qb)], n, G, kvr)


@pytest.mark.parametrize("n", [(1 << 23) - 1, (1 << 23) + 5, (1 << 24) + 77])
def test_rows_beyond_the_range_of_a_byte_offset(program, n):
    """Heads so long that 256 times the rows left to the end does not fit 31 bits."""
    nqb = -(-n // 256)
    for qb in (0, 1):
        waves = run_workgroup(program, n, 2, 1, (1, qb), None, nqb)
        check_workgroup(waves, [(1, qb)], n, 2, 1)


@pytest.mark.parametrize("n,rounds,vid0,kvr", [(513, 4, 0, 1), (600, 6, 31, 2), (700, 4, 2, 1), (1000, 4, 33, 4), (1024, 4, 35, 1),
                                               (1537, 6, 70, 5), (2000, 4, 5, 1), (3001, 2, 7, 4), (3001, 4, 11, 1)])
@pytest.mark.parametrize("seed", [None, 3])
def test_pairs_of_blocks(program, n, rounds, vid0, kvr, seed):
    nqb = -(-n // 256)
    blocks = pair_blocks(vid0, rounds, nqb)
    G = max(g for g, _ in blocks) + 1          # the last head of the tensor is among them
    waves = run_workgroup(program, n, G, kvr, blocks[0], None, nqb, seed=seed, rounds=rounds, vid0=vid0)
    check_workgroup(waves, blocks, n, G, kvr)


def test_catches_an_unclamped_tile(program):
    """Planted mistake: the partial tile is fetched whole."""
    prog, labels = program
    bad = [("s_nop", ["0"]) if op == "v_min_u32" and a[2] != "%[qoff]" else (op, a) for op, a in prog]
    waves = run_workgroup((bad, labels), 600, 1, 1, (0, 2), None, 3)
    with pytest.raises(AssertionError):
        check_workgroup(waves, [(0, 2)], 600, 1, 1)


def test_catches_offsets_that_stay_clamped(program):
    """Planted mistake: the lane offsets are not restored after the partial tile."""
    prog, labels = program
    bad = list(prog)
    for name, at in labels.items():
        if name.startswith("Lfa"):
            for i in range(4):
                assert bad[at + i][0] == "v_add_u32"
    outside = [i for i, (op, a) in enumerate(prog) if op == "v_add_u32" and a[2] in ("%[kl0]", "%[vl0]")][8:]
    for i in outside:
        bad[i] = ("s_nop", ["0"])
    blocks = pair_blocks(0, 4, 3)
    waves = run_workgroup((bad, labels), 700, 24, 1, blocks[0], None, 3, rounds=4, vid0=0)
    with pytest.raises(AssertionError):
        check_workgroup(waves, blocks, 700, 24, 1)


def test_catches_a_store_past_the_rows(program):
    """Planted mistake: the stores keep the full execution mask."""
    prog, labels = program
    bad = [(op, [a[0], "0x7fffffff", a[2]]) if op == "v_cmpx_gt_i32" else (op, a) for op, a in prog]
    waves = run_workgroup((bad, labels), 600, 1, 1, (0, 2), None, 3)
    with pytest.raises(AssertionError):
        check_workgroup(waves, [(0, 2)], 600, 1, 1)
