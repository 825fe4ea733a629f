"""Software wait states in the built device code (CPU only).

gfx950 does not wait by itself for some results: a matrix product's, for instance, has to be left alone for eight (bf16,
16x16x32 and 16x16x16) or ten (fp32, 16x16x4) wait states, an instruction or s_nop step each.  The compiler puts them in,
but (ROCm 7.2) counts them along one path to a join of branches only, through the code that the other path jumps over: a
use behind the join can come too early on the other.  So every path of every kernel is followed here.

The rules are the ones that the compiler keeps in straight code; a product's result as accumulator of the next product of
its kind, in the same registers, needs none."""
import os
import re
import struct
import subprocess

import pytest

from test_abi_host import LIB, pf  # noqa: F401  (fixture: builds / loads the library)

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# matrix instruction: wait states until its result may be read or overwritten, until its accumulator operand may be overwritten
PRODUCTS = {"v_mfma_f32_16x16x32_bf16": (8, 3), "v_mfma_f32_16x16x16_bf16": (8, 3), "v_mfma_f32_16x16x4_f32": (10, 0)}
TRANS = ("v_exp_", "v_log_", "v_rcp_", "v_rsq_", "v_sqrt_", "v_sin_", "v_cos_")
MEMORY = ("ds_", "global_", "buffer_", "flat_", "scratch_")
NO_RESULT = ("ds_write", "ds_append", "global_store", "buffer_store", "flat_store", "scratch_store", "global_load_lds", "buffer_wb", "buffer_inv")
REG = re.compile(r"(?<![\w.])([vas])(?:(\d+)|\[(\d+):(\d+)\])(?!\w)|(?<!\w)(vcc|exec)(?!\w)")


def _regs(text):
    out = []
    for k, one, lo, hi, name in REG.findall(text):
        out += [name] if name else [k + str(i) for i in range(int(one or lo), int(one or hi) + 1)]
    return out


class Instr:
    """op, registers written, read; of products: operands a and b in read, accumulator apart."""

    def __init__(self, text):
        self.text = text
        self.op, _, rest = text.partition(" ")
        o = [_regs(p) for p in re.split(r",(?![^\[]*\])", rest)]
        flat = lambda parts: [r for p in parts for r in p]
        self.acc, self.product = [], self.op in PRODUCTS
        self.valu = self.op.startswith("v_") and not self.product
        if self.op.startswith("v_mfma") and not self.product:
            raise AssertionError("no rule for " + text)
        if not self.op.startswith(("v_",) + MEMORY):
            self.write, self.read = [], []
        elif self.product:
            self.write, self.read, self.acc = o[0], o[1] + o[2], o[3]
        elif self.op.startswith(NO_RESULT) or (self.op.startswith(MEMORY) and " lds" in text):
            self.write, self.read = [], flat(o)
        else:
            two = re.match(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[ui]64", self.op) is not None
            self.write, self.read = flat(o[:1 + two]), flat(o[1 + two:])
            if re.search(r"fmac|dot\w*c_|swap|writelane|_dpp|d16", self.op):
                self.read = self.read + o[0]
        self.dpp = "dpp" in self.op or "row_" in text or "quad_perm" in text


def _functions(listing):
    name, body, labels = None, [], {}
    for line in listing.splitlines():
        m = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
        if m and re.fullmatch(r"L\d+", m.group(1)):
            labels[m.group(1)] = len(body)
        elif m:
            if body:
                yield name, body, labels
            name, body, labels = m.group(1), [], {}
        elif name and line.startswith("\t"):
            text = line.split("//")[0].strip()
            if text:
                body.append(text)
    if body:
        yield name, body, labels


def missing_waits(body, labels):
    """{(index of the early use, of the producer): wait states missing}, the worst over all paths."""
    ins, n = [Instr(t) for t in body], len(body)
    ends = {i + 1 for i in range(n) if ins[i].op.startswith(("s_cbranch", "s_branch", "s_endpgm"))}
    starts = sorted(({0} | set(labels.values()) | ends) - {n})
    stop = dict(zip(starts, starts[1:] + [n]))
    entry, todo, found = {0: {}}, [0], {}
    while todo:
        first = todo.pop()
        # what is under way: (rule, register) -> (time from which it may be used, producer); time is counted from `first`
        busy, t = dict(entry[first]), 0

        def use(i, rule, regs):
            for r in regs:
                ready, by = busy.get((rule, r), (0, 0))
                if ready > t:
                    found[i, by] = max(found.get((i, by), 0), ready - t)

        for i in range(first, stop[first]):
            x = ins[i]
            if x.product:
                use(i, "result", x.read)
                use(i, "valu", x.read + x.acc)
                for r in x.acc:
                    ready, by = busy.get(("result", r), (0, 0))
                    if ready > t and not (ins[by].write == x.acc and PRODUCTS[ins[by].op] == PRODUCTS[x.op]):
                        found[i, by] = max(found.get((i, by), 0), ready - t)
            elif x.valu:
                use(i, "result", x.read + x.write)
                use(i, "accumulator", x.write)
                use(i, "sgpr", x.read)
                use(i, "dpp", x.read if x.dpp else [])
                use(i, "lane", x.read if x.op.startswith("v_readlane") or x.op.startswith("v_readfirstlane") else [])
                use(i, "trans", x.read if not x.op.startswith(TRANS) else [])
            elif x.op.startswith(MEMORY):
                use(i, "result", x.read)
                use(i, "address", x.read)
            t += int(x.text.split()[1], 0) + 1 if x.op == "s_nop" else 1
            for r in x.write:
                if x.product or x.valu:
                    for rule in ("result", "valu", "dpp", "lane", "trans", "sgpr", "address"):
                        busy.pop((rule, r), None)
                if x.product:
                    busy["result", r] = (t + PRODUCTS[x.op][0], i)
                elif x.valu:
                    rules = (("sgpr", 2), ("address", 5)) if r[0] == "s" or r in ("vcc", "exec") else (("valu", 2), ("dpp", 2), ("lane", 1))
                    for rule, wait in rules + ((("trans", 1),) if x.op.startswith(TRANS) else ()):
                        busy[rule, r] = (t + wait, i)
            for r in x.acc:
                busy["accumulator", r] = (t + PRODUCTS[x.op][1], i)
        last = ins[stop[first] - 1]
        after = []
        if last.op.startswith(("s_cbranch", "s_branch")):
            after.append(labels[last.text.split()[1].strip("<>")])
        elif last.op.startswith(("s_setpc", "s_swappc")):
            raise AssertionError("a call: " + last.text)
        if last.op not in ("s_branch", "s_endpgm") and stop[first] < n:
            after.append(stop[first])
        out = {k: (ready - t, by) for k, (ready, by) in busy.items() if ready > t}
        for s in after:
            known = entry.get(s)
            if known is None:
                entry[s] = dict(out)
                todo.append(s)
                continue
            worse = {k: v for k, v in out.items() if v[0] > known.get(k, (0, 0))[0]}
            if worse:
                known.update(worse)
                if s not in todo:
                    todo.append(s)
    return found


def _listings(tmp_path):
    data, at, k = open(LIB, "rb").read(), 0, 0
    while True:
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)
        if at < 0:
            return
        (entries,), p = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            if size and b"gfx950" in data[p + 24:p + 24 + length]:
                path = tmp_path / f"{k}.co"
                path.write_bytes(data[at + offset:at + offset + size])
                yield subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--symbolize-operands", str(path)], check=True,
                                     capture_output=True, text=True).stdout
                k += 1
            p += 24 + length
        at += 1


JOIN = """0 <kernel>:
\tv_mfma_f32_16x16x4_f32 v[2:5], v2, v3, 0
\ts_cbranch_scc1 L0
{between}
10 <L0>:
{after}
\tv_mul_f32_e32 v5, s4, v5
\ts_endpgm
"""
MOVE = "\tv_mov_b32_e32 v9, s4\n"


@pytest.mark.parametrize("between,after,missing", [(9, 0, 9), (3, 6, 3), (9, 9, 0), (0, 8, 1)])
def test_the_shorter_path_decides(between, after, missing):
    (_, body, labels), = _functions(JOIN.format(between=MOVE * between, after=MOVE * after))
    assert list(missing_waits(body, labels).values()) == ([missing] if missing else [])


@pytest.mark.parametrize("lines,missing", [
    (["v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], 0", "v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], v[0:3]"], 0),
    (["v_mfma_f32_16x16x32_bf16 v[0:3], v[8:11], v[12:15], 0", "s_nop 6", "ds_write_b128 v20, v[0:3]"], 1),
    (["v_mfma_f32_16x16x32_bf16 a[0:3], v[8:11], v[12:15], v[4:7]", "s_nop 1", "v_mov_b32_e32 v5, v30"], 1),
    (["v_mov_b32_e32 v1, v2", "s_nop 0", "v_fmac_f32_dpp v3, -v1, v4 row_newbcast:3 row_mask:0xf bank_mask:0xf"], 1),
    (["v_readfirstlane_b32 s4, v2", "s_nop 3", "global_load_dwordx4 v[4:7], v8, s[4:5]"], 1),
    (["v_cmp_gt_f32_e32 vcc, v1, v2", "s_nop 1", "v_cndmask_b32_e32 v3, v4, v5, vcc"], 0)])
def test_rules(lines, missing):
    (_, body, labels), = _functions("0 <kernel>:\n" + "".join(f"\t{x}\n" for x in lines + ["s_endpgm"]))
    assert sum(missing_waits(body, labels).values()) == missing


def test_no_kernel_uses_a_result_too_early(pf, tmp_path):  # noqa: F811
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    kernels = 0
    for listing in _listings(tmp_path):
        for name, body, labels in _functions(listing):
            kernels += any(t.startswith("v_mfma") for t in body)
            early = missing_waits(body, labels)
            assert not early, (name, [(body[by], body[i], w) for (i, by), w in list(early.items())[:4]])
    assert kernels > 100


def test_no_kernel_keeps_registers_in_memory(pf, tmp_path):  # noqa: F811
    """Neither spills nor arrays that the compiler left in scratch memory."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    for listing in _listings(tmp_path):
        for name, body, _ in _functions(listing):
            assert not [t for t in body if t.startswith("scratch_")], name
