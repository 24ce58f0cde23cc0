"""Address simulation of one wave of a kernel of this library, from the assembly that hipcc writes for it.

Integer instructions are executed for all 64 lanes; floating-point and matrix results are taken as zero, except in the
compiler's integer division.  Memory holds no data, only bounds: a load has to lie in one of the given buffers.  The vector
memory counter and LDS are followed as far as a ring of direct global -> LDS loads needs it:

  * a word of LDS may be read only when the direct load that wrote it last has landed (the wave's own `s_waitcnt vmcnt`);
  * it may be requested again only when the reads of it have returned (`s_waitcnt lgkmcnt`).

The simulation ends at the first barrier (or the end of the kernel): up to there a wave's LDS region is its own.
An instruction that is not known here is an error, so that nothing is skipped silently."""
import re
import struct
from collections import deque

import numpy as np

M32, M64 = 0xFFFFFFFF, 0xFFFFFFFFFFFFFFFF
KERNARG = 0x1000
LANES = np.arange(64, dtype=np.uint64)


class Fault(Exception):
    pass


def kernels(text):
    """{mangled name: its lines} of an assembly file."""
    out = {}
    for m in re.finditer(r"^(_ZN\S+):", text, re.M):
        end = text.find(".Lfunc_end", m.end())
        out[m.group(1)] = text[m.end():end].split("\n")
    return out


def metadata(text):
    """{mangled name: {key: number}} of the kernels' resource figures (.vgpr_spill_count and the like)."""
    out = {}
    for block in text[text.index("amdhsa.kernels:"):].split("  - .agpr_count")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        out[name] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\s*$", block, re.M)}
    return out


class Instr:
    __slots__ = ("op", "args", "mods", "text", "asm")

    def __init__(self, op, args, mods, text, asm):
        self.op, self.args, self.mods, self.text, self.asm = op, args, mods, text, asm


def program(lines):
    """(instructions, {label: index}); Instr.asm: written by hand (an asm statement of the source)."""
    code, labels, asm = [], {}, False
    for line in lines:
        if "#ASMSTART" in line or "#ASMEND" in line:
            asm = "#ASMSTART" in line
        line = line.split(";")[0].strip()
        m = re.match(r"^(\.L\w+):", line)
        if m:
            labels[m.group(1)] = len(code)
            continue
        if not line or line.startswith("."):
            continue
        op, _, rest = line.partition(" ")
        mods = {k: int(v, 0) for k, v in re.findall(r"\b(offset|offset0|offset1|bitop3):(\S+)", rest)}
        rest = re.sub(r"\b[a-z]\w*:(\[[^]]*\]|[\w.]+)", "", rest)
        code.append(Instr(re.sub(r"_(e32|e64|sdwa)$", "", op), [a.strip() for a in rest.split(",")] if rest.strip() else [],
                          mods, line, asm))
    return code, labels


def _signed(v, bits=32):
    v &= (1 << bits) - 1
    return v - (1 << bits) if v >> (bits - 1) else v


_CMP = {"eq": lambda x, y: x == y, "ne": lambda x, y: x != y, "lg": lambda x, y: x != y, "gt": lambda x, y: x > y,
        "ge": lambda x, y: x >= y, "lt": lambda x, y: x < y, "le": lambda x, y: x <= y}
_BIT = {"and": lambda x, y: x & y, "or": lambda x, y: x | y, "xor": lambda x, y: x ^ y, "andn2": lambda x, y: x & ~y}


def _i(v):
    return v.astype(np.uint32).view(np.int32).astype(np.int64)


# vector operations on uint64 arrays that hold 32-bit values; the result is cut to 32 bits
_VOP = {
    "v_and_b32": lambda x, y: x & y, "v_or_b32": lambda x, y: x | y, "v_xor_b32": lambda x, y: x ^ y,
    "v_add_u32": lambda x, y: x + y, "v_sub_u32": lambda x, y: x - y, "v_subrev_u32": lambda x, y: y - x,
    "v_lshlrev_b32": lambda x, y: y << (x & 31), "v_lshrrev_b32": lambda x, y: y >> (x & 31),
    "v_ashrrev_i32": lambda x, y: (_i(y) >> (x & 31).astype(np.int64)).astype(np.uint64),
    "v_mul_lo_u32": lambda x, y: x * y, "v_mul_hi_u32": lambda x, y: (x * y) >> 32,
    "v_mul_u32_u24": lambda x, y: (x & 0xFFFFFF) * (y & 0xFFFFFF),
    "v_mul_i32_i24": lambda x, y: (((_i(x) << 40 >> 40)) * (_i(y) << 40 >> 40)).astype(np.uint64),
    "v_min_u32": np.minimum, "v_max_u32": np.maximum,
    "v_min_i32": lambda x, y: np.minimum(_i(x), _i(y)).astype(np.uint64),
    "v_max_i32": lambda x, y: np.maximum(_i(x), _i(y)).astype(np.uint64),
    "v_lshl_add_u32": lambda x, y, z: (x << (y & 31)) + z, "v_add_lshl_u32": lambda x, y, z: (x + y) << (z & 31),
    "v_lshl_or_b32": lambda x, y, z: (x << (y & 31)) | z, "v_and_or_b32": lambda x, y, z: (x & y) | z,
    "v_or3_b32": lambda x, y, z: x | y | z, "v_add3_u32": lambda x, y, z: x + y + z, "v_xad_u32": lambda x, y, z: (x ^ y) + z,
    "v_bfe_u32": lambda x, y, z: (x >> (y & 31)) & ((np.uint64(1) << (z & 31)) - 1),
    "v_med3_i32": lambda x, y, z: np.sort(np.stack([_i(x), _i(y), _i(z)]), axis=0)[1].astype(np.uint64),
    "v_alignbit_b32": lambda x, y, z: ((x << 32) | y) >> (z & 31),
    "v_mov_b32": lambda x: x,
}
# results that no address depends on
_ZERO = re.compile(r"v_(mfma|cvt_|fma|fmac|perm|mul_f|add_f|max_f|bfe_i32)")
_LOAD = {"global_load_dword": 4, "global_load_dwordx2": 8, "global_load_dwordx4": 16, "global_load_ushort": 2}
_DS = {"ds_read_b128": 16, "ds_read_b64": 8, "ds_read_b32": 4, "ds_read_u16": 2}


class DirectLoad:
    """A direct global -> LDS load: buffer, per-lane byte offset in it, LDS address of lane 0, bytes per lane, when."""

    def __init__(self, buf, off, lds, size, at):
        self.buf, self.off, self.lds, self.size, self.at, self.landed = buf, off, lds, size, at, False


class Wave:
    """One wave: run() returns its direct loads in order.  buffers: {name: (address, bytes)}; lds_bytes: its workgroup's."""

    def __init__(self, prog, kernarg, workgroup, wave, buffers, lds_bytes, limit=300000):
        self.code, self.labels = prog
        self.kernarg, self.buffers, self.limit = kernarg, buffers, limit
        self.s, self.v = [0] * 128, np.zeros((512, 64), np.uint64)
        self.st = {"vcc": 0, "exec": M64, "m0": 0, "scc": 0}
        self.s[0], self.s[2] = KERNARG, workgroup
        self.v[0] = LANES + np.uint64(64 * wave)
        self.loads, self.vm, self.lgkm = [], deque(), deque()
        self.own_waits = []                                           # when the compiler's own code waited for loads
        self.word = np.full(lds_bytes // 4, -1, np.int64)            # direct load that wrote (or will write) a word of LDS
        self.busy = np.zeros(lds_bytes // 4, np.int32)               # reads of the word that have not returned
        self.seen = np.zeros(lds_bytes // 4, bool)                   # the word has been read since

    # ---- operands -----------------------------------------------------------------------------------------------
    def _reg(self, o):
        m = re.match(r"^([sv])(?:(\d+)|\[(\d+):(\d+)\])$", o)
        return (m.group(1), int(m.group(2) or m.group(3))) if m else None

    def sget(self, o, bits=32):
        if o in self.st:
            return self.st[o] & (M64 if bits == 64 else M32)
        if o in ("vcc_lo", "vcc_hi"):
            return self.st["vcc"] >> (32 if o == "vcc_hi" else 0) & M32
        r = self._reg(o)
        if r and r[0] == "s":
            return self.s[r[1]] | (self.s[r[1] + 1] << 32 if bits == 64 else 0)
        if r:                                                         # (v_readfirstlane)
            return int(self.v[r[1], self._first()])
        if re.match(r"^-?(\d+|0x[0-9a-f]+)$", o):
            return int(o, 0) & (M64 if bits == 64 else M32)
        if re.match(r"^-?\d*\.\d+$", o):
            return struct.unpack("<I", struct.pack("<f", float(o)))[0]
        raise Fault(f"operand {o}")

    def sput(self, o, val, bits=32):
        if o in self.st:
            self.st[o] = val & (M64 if o != "m0" else M32)
            return
        r = self._reg(o)
        if not r or r[0] != "s":
            raise Fault(f"destination {o}")
        self.s[r[1]] = val & M32
        if bits == 64:
            self.s[r[1] + 1] = val >> 32 & M32

    def vget(self, o, bits=32):
        r = self._reg(o)
        if r and r[0] == "v":
            return self.v[r[1]] | (self.v[r[1] + 1] << np.uint64(32)) if bits == 64 else self.v[r[1]]
        return np.full(64, self.sget(o, bits), np.uint64)

    def vput(self, o, val, bits=32):
        n, on = self._reg(o)[1], self._lanes(self.st["exec"])
        self.v[n] = np.where(on, val & np.uint64(M32), self.v[n])
        if bits == 64:
            self.v[n + 1] = np.where(on, val >> np.uint64(32), self.v[n + 1])

    def _lanes(self, mask):
        return np.full(64, mask == M64) if mask in (0, M64) else (np.uint64(mask) >> LANES & np.uint64(1)) != 0

    def _mask(self, flags):
        return int(np.packbits(flags, bitorder="little").view(np.uint64)[0]) & self.st["exec"]

    def _first(self):
        return (self.st["exec"] & -self.st["exec"]).bit_length() - 1 if self.st["exec"] else 0

    # ---- memory -------------------------------------------------------------------------------------------------
    def _inside(self, addr, size, text):
        """(names, offsets): the buffers that the addresses lie in, joined by +, and the offsets in them."""
        names, off = [], np.full(len(addr), M64, np.uint64)
        for name, (base, n) in self.buffers.items():
            here = (addr >= np.uint64(base)) & (addr <= np.uint64(base + n - size))
            if here.any():
                names.append(name)
                off[here] = addr[here] - np.uint64(base)
        if (off == np.uint64(M64)).any():
            raise Fault(f"out of bounds: {int(addr[off == np.uint64(M64)][0]):#x} ({text})")
        return "+".join(names), off

    def _address(self, voff, sbase, mods):
        a = self.vget(voff, 64) if sbase == "off" else self.vget(voff) + np.uint64(self.sget(sbase, 64))
        return a + np.uint64(mods.get("offset", 0) & M64)

    def _direct(self, i, size):
        on = self._lanes(self.st["exec"])
        if not on.any():
            return
        addr = self._address(i.args[0], i.args[1], i.mods)
        name, inside = self._inside(addr[on], size, i.text)
        off = np.full(64, M64, np.uint64)
        off[on] = inside
        m0 = self.st["m0"]
        ld = DirectLoad(name, off, m0, size, self.steps)
        words = np.concatenate([np.arange((m0 + size * l) // 4, (m0 + size * (l + 1)) // 4) for l in range(64) if on[l]]) \
            if not on.all() else np.arange(m0 // 4, (m0 + 64 * size) // 4)
        if words[-1] >= len(self.word):
            raise Fault(f"beyond LDS ({i.text})")
        if self.busy[words].any():
            raise Fault(f"requested again before the reads have returned ({i.text})")
        old = self.word[words]
        for n in np.unique(old[old >= 0]):
            if not self.loads[n].landed:
                raise Fault(f"requested again before it has landed ({i.text})")
            if self.loads[n].buf in ("Xq", "Wq") and not self.seen[words[old == n]].all():
                raise Fault(f"requested again before it was read ({i.text})")
        self.word[words], self.seen[words] = len(self.loads), False
        self.vm.append(ld)
        self.loads.append(ld)

    def _ds_read(self, i):
        step = {"ds_read2_b64": 8, "ds_read2_b32": 4, "ds_read2st64_b32": 256}.get(i.op)
        size = _DS.get(i.op) or min(step, 8 if i.op.endswith("b64") else 4)
        offs = [i.mods.get("offset", 0)] if step is None else [step * i.mods.get("offset0", 0), step * i.mods.get("offset1", 0)]
        base, on = self.vget(i.args[1]), self._lanes(self.st["exec"])
        words = np.unique(np.concatenate([(base[on] + np.uint64(o + b) & np.uint64(M32)) // np.uint64(4)      # (32-bit sums)
                                          for o in offs for b in range(0, size, 4)]))
        words = words.astype(np.int64)
        if len(words) and words[-1] >= len(self.word):
            raise Fault(f"beyond LDS ({i.text})")
        for n in np.unique(self.word[words]):
            if n < 0 or not self.loads[n].landed:
                raise Fault(f"read before it has landed ({i.text})")
        self.busy[words] += 1
        self.seen[words] = True
        self.lgkm.append(words)
        self._zero(i.args[0])

    def _zero(self, o):
        m = re.match(r"^v\[(\d+):(\d+)\]$", o)
        a, b = (int(m.group(1)), int(m.group(2))) if m else (int(o[1:]),) * 2
        self.v[a:b + 1] = 0

    def _wait(self, text):
        m = re.search(r"vmcnt\((\d+)\)", text)
        if m:
            while len(self.vm) > int(m.group(1)):
                ld = self.vm.popleft()
                if ld is not None:
                    ld.landed = True
        m = re.search(r"lgkmcnt\((\d+)\)", text)
        if m:
            while len(self.lgkm) > int(m.group(1)):
                words = self.lgkm.popleft()
                if words is not None:
                    self.busy[words] -= 1

    # ---- the run ------------------------------------------------------------------------------------------------
    def run(self):
        pc, self.steps = 0, 0
        while True:
            i = self.code[pc]
            pc += 1
            self.steps += 1
            if self.steps > self.limit:
                raise Fault("no end")
            if i.op in ("s_barrier", "s_endpgm"):
                break
            if i.op == "s_branch":
                pc = self.labels[i.args[0]]
            elif i.op.startswith("s_cbranch"):
                st = self.st
                if {"scc0": not st["scc"], "scc1": st["scc"], "vccz": not st["vcc"], "vccnz": st["vcc"],
                        "execz": not st["exec"], "execnz": st["exec"]}[i.op[10:]]:
                    pc = self.labels[i.args[0]]
            else:
                try:
                    (self._scalar if i.op[0] == "s" else self._vector)(i)
                except Fault as e:
                    raise Fault(f"{e} at instruction {pc} after {self.steps}") from None
        live = self.word[self.word >= 0]
        for n in np.unique(live):
            if not self.loads[n].landed:
                raise Fault("a direct load is still under way at the barrier")
            if self.loads[n].buf in ("Xq", "Wq") and not self.seen[self.word == n].all():
                raise Fault("a direct load was never read")
        return self.loads

    def _scalar(self, i):
        op, a, st = i.op, i.args, self.st
        if op == "s_waitcnt":
            if "vmcnt" in i.text and not i.asm:
                self.own_waits.append(self.steps)
            return self._wait(i.text)
        if op in ("s_nop", "s_setprio", "s_sleep"):
            return None
        if op.startswith("scratch_"):
            self.vm.append(None)
            return self._zero(a[0]) if op.startswith("scratch_load") else None
        if op.startswith("s_load_dword"):
            addr, reg = self.sget(a[1], 64) + int(a[2], 0), self._reg(a[0])[1]
            self.lgkm.append(None)
            for n in range(int(op[13:] or 1)):
                where = addr + 4 * n - KERNARG
                if 0 <= where <= len(self.kernarg) - 4:
                    self.s[reg + n] = struct.unpack_from("<I", self.kernarg, where)[0]
                else:
                    self._inside(np.array([addr + 4 * n], np.uint64), 4, i.text)
                    self.s[reg + n] = 0
            return None
        m = re.match(r"s_cmpk?_(eq|lg|gt|ge|lt|le)_(i32|u32|u64)$", op)
        if m:
            bits = 64 if m.group(2) == "u64" else 32
            x, y = self.sget(a[0], bits), self.sget(a[1], bits)
            if m.group(2) == "i32":
                x, y = _signed(x), _signed(y)
            st["scc"] = int(_CMP[m.group(1)](x, y))
            return None
        m = re.match(r"s_bitcmp([01])_b32$", op)
        if m:
            st["scc"] = int((self.sget(a[0]) >> (self.sget(a[1]) & 31) & 1) == int(m.group(1)))
            return None
        m = re.match(r"s_(and|or|andn2)_saveexec_b64$", op)
        if m:
            x, e = self.sget(a[1], 64), st["exec"]
            self.sput(a[0], e, 64)
            st["exec"] = _BIT[m.group(1)](x, e) & M64
            st["scc"] = int(st["exec"] != 0)
            return None
        m = re.match(r"s_(and|or|xor|andn2)_b(32|64)$", op)
        if m:
            bits = int(m.group(2))
            val = _BIT[m.group(1)](self.sget(a[1], bits), self.sget(a[2], bits)) & (M64 if bits == 64 else M32)
            st["scc"] = int(val != 0)
            return self.sput(a[0], val, bits)
        m = re.match(r"s_(lshl|lshr|ashr)_([bi])(32|64)$", op)
        if m:
            bits = int(m.group(3))
            x, n = self.sget(a[1], bits), self.sget(a[2]) & (bits - 1)
            x = x << n if m.group(1) == "lshl" else (_signed(x, bits) if m.group(1) == "ashr" else x) >> n
            x &= M64 if bits == 64 else M32
            st["scc"] = int(x != 0)
            return self.sput(a[0], x, bits)
        m = re.match(r"s_cselect_b(32|64)$", op)
        if m:
            return self.sput(a[0], self.sget(a[1] if st["scc"] else a[2], int(m.group(1))), int(m.group(1)))
        m = re.match(r"s_mov_b(32|64)$", op)
        if m:
            return self.sput(a[0], self.sget(a[1], int(m.group(1))), int(m.group(1)))
        if op in ("s_movk_i32", "s_mulk_i32", "s_addk_i32"):
            k = _signed(int(a[1], 0), 16) if int(a[1], 0) > 0 else int(a[1], 0)
            x = _signed(self.sget(a[0]))
            val = k if op == "s_movk_i32" else x * k if op == "s_mulk_i32" else x + k
            if op == "s_addk_i32":
                st["scc"] = int(not -2 ** 31 <= val < 2 ** 31)
            return self.sput(a[0], val)
        if op in ("s_not_b32", "s_abs_i32"):
            x = self.sget(a[1])
            val = ~x & M32 if op == "s_not_b32" else abs(_signed(x)) & M32
            st["scc"] = int(val != 0)
            return self.sput(a[0], val)
        x, y = self.sget(a[1]), self.sget(a[2])
        if op in ("s_add_u32", "s_addc_u32"):
            val = x + y + (st["scc"] if op == "s_addc_u32" else 0)
            st["scc"] = val >> 32
        elif op in ("s_sub_u32", "s_subb_u32"):
            y += st["scc"] if op == "s_subb_u32" else 0
            val, st["scc"] = x - y, int(y > x)
        elif op in ("s_add_i32", "s_sub_i32"):
            val = _signed(x) + (_signed(y) if op == "s_add_i32" else -_signed(y))
            st["scc"] = int(not -2 ** 31 <= val < 2 ** 31)
        elif op == "s_mul_i32":
            val = x * y
        elif op == "s_mul_hi_u32":
            val = x * y >> 32
        elif op == "s_mul_hi_i32":
            val = _signed(x) * _signed(y) >> 32
        elif op in ("s_min_i32", "s_max_i32", "s_min_u32", "s_max_u32"):
            x, y = (_signed(x), _signed(y)) if op.endswith("i32") else (x, y)
            val = min(x, y) if op[2:5] == "min" else max(x, y)
            st["scc"] = int(val == x)
        elif op == "s_bfe_u32":
            val = x >> (y & 31) & ((1 << (y >> 16 & 127)) - 1)
            st["scc"] = int(val != 0)
        else:
            raise Fault(f"unknown: {i.text}")
        return self.sput(a[0], val & M32)

    def _vector(self, i):
        op, a = i.op, i.args
        if op in _VOP:
            return self.vput(a[0], _VOP[op](*[self.vget(o) for o in a[1:]]) & np.uint64(M32))
        if op == "global_load_lds_dwordx4":
            return self._direct(i, 16)
        if op == "global_load_lds_dword":
            return self._direct(i, 4)
        if op in _LOAD:
            on = self._lanes(self.st["exec"])
            if on.any():
                self._inside(self._address(a[1], a[2], i.mods)[on], _LOAD[op], i.text)
                self.vm.append(None)
            return self._zero(a[0])
        if op.startswith("ds_read"):
            return self._ds_read(i)
        if op.startswith("ds_write"):                                 # (the partial tile takes the ring's place)
            return self.lgkm.append(None)
        if op == "v_readfirstlane_b32":
            return self.sput(a[0], self.sget(a[1]))
        if op == "v_mov_b64":
            return self.vput(a[0], self.vget(a[1], 64), 64)
        if op == "v_cndmask_b32":
            return self.vput(a[0], np.where(self._lanes(self.sget(a[3], 64)), self.vget(a[2]), self.vget(a[1])))
        m = re.match(r"v_cmp_(eq|ne|gt|ge|lt|le)_(i32|u32|u64)$", op)
        if m:
            bits = 64 if m.group(2) == "u64" else 32
            x, y = self.vget(a[1], bits), self.vget(a[2], bits)
            if m.group(2) == "i32":
                x, y = _i(x), _i(y)
            return self.sput(a[0], self._mask(_CMP[m.group(1)](x, y)), 64)
        if op == "v_lshlrev_b64":
            return self.vput(a[0], self.vget(a[2], 64) << (self.vget(a[1]) & np.uint64(63)), 64)
        if op == "v_lshl_add_u64":
            return self.vput(a[0], (self.vget(a[1], 64) << (self.vget(a[2]) & np.uint64(63))) + self.vget(a[3], 64), 64)
        if op == "v_mad_u64_u32":
            return self.vput(a[0], self.vget(a[2]) * self.vget(a[3]) + self.vget(a[4], 64), 64)
        if op == "v_mad_i64_i32":
            return self.vput(a[0], (_i(self.vget(a[2])) * _i(self.vget(a[3]))).astype(np.uint64) + self.vget(a[4], 64), 64)
        if op == "v_bitop3_b32":
            x, y, z = (self.vget(o) for o in a[1:4])
            val = np.zeros(64, np.uint64)
            for n in range(8):
                if i.mods["bitop3"] >> n & 1:
                    val |= (x if n & 4 else ~x) & (y if n & 2 else ~y) & (z if n & 1 else ~z)
            return self.vput(a[0], val & np.uint64(M32))
        # the integer division of the compiler (a uniform one: all lanes alike)
        if op == "v_cvt_f32_u32":
            return self.vput(a[0], self.vget(a[1]).astype(np.float32).view(np.uint32).astype(np.uint64))
        if op in ("v_rcp_iflag_f32", "v_mul_f32", "v_cvt_u32_f32"):
            f = [self.vget(o).astype(np.uint32).view(np.float32).astype(np.float64) for o in a[1:]]
            if op == "v_cvt_u32_f32":
                return self.vput(a[0], np.clip(f[0], 0, M32).astype(np.uint64))
            with np.errstate(divide="ignore"):
                val = 1.0 / f[0] if op == "v_rcp_iflag_f32" else f[0] * f[1]
            return self.vput(a[0], val.astype(np.float32).view(np.uint32).astype(np.uint64))
        if _ZERO.match(op):
            return self._zero(a[0])
        raise Fault(f"unknown: {i.text}")
