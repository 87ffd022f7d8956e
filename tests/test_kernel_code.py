"""What the compiler made of the kernels that depend on its scheduling, read
from the disassembly of the library built here (CPU only)."""
import os
import re
import shutil
import subprocess

import pytest

import paper_1801_01072_amd as ent

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
pytestmark = pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(ent.LIB_PATH),
                                reason="needs llvm-objdump and the built library")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Mangled name -> instructions (address, mnemonic, operands) of every
    kernel of the dense and BF16x3 code objects."""
    d = tmp_path_factory.mktemp("code")
    lib = str(d / "lib.so")
    shutil.copy(ent.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, capture_output=True)
    out = {}
    for f in sorted(d.glob("lib.so.*gfx950*")):
        syms = subprocess.run([OBJDUMP, "-t", str(f)], capture_output=True, text=True, check=True).stdout
        if "batch_dense_" not in syms and "batch_bf16x3_" not in syms:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True,
                              check=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\S+)>:$", line)
            if m:
                name = m.group(1)
                out[name] = []
                continue
            m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):?", line)
            if m and name:
                out[name].append((int(m.group(3), 16), m.group(1), m.group(2)))
    return out


def test_dense_k_loops_wait_only_where_they_say(kernels):
    """The K loop of a dense tile keeps two chunks of direct loads to LDS in
    flight: its own waits for them stand ahead of a barrier.  A wait for loads
    straight ahead of an LDS read is the compiler's, and drains them all."""
    names = [n for n in kernels if re.search(r"(batch_dense_step|batch_dense_persistent|dense_step|dense_step_split)_kernel", n)
             and any(op.startswith("global_load_lds") for _, op, _ in kernels[n])]
    assert len(names) >= 16
    for n in names:
        ins = kernels[n]
        bad = [hex(a) for i, (a, op, args) in enumerate(ins) if op == "s_waitcnt" and "vmcnt(0)" in args
               and any(o.startswith("ds_read") for _, o, _ in ins[i + 1:i + 3])]
        assert not bad, (n, bad)


def exec_at_barriers(ins):
    """Addresses of the barriers that some path reaches with part of the wave's
    lanes masked off.  Masks are followed symbolically through the scalar registers,
    path by path: ALL, (sub, mask, id): some lanes of a mask, (diff, mask, id): its
    others, ANY: not known."""
    index = {a: i for i, (a, _, _) in enumerate(ins)}
    ALL, ANY = ("all",), ("any",)

    def either(x, y):
        if ALL in (x, y) or x == y:
            return x if x == y else ALL
        for p, q in ((x, y), (y, x)):
            if p[0] == "sub" and q[0] == "diff" and p[1:] == q[1:]:
                return p[1]
            if p[0] in ("sub", "diff") and p[1] == q:
                return q
        return ANY

    def without(x, y):  # x & ~y, y part of x
        if y[0] in ("sub", "diff") and y[1] == x:
            return ("diff" if y[0] == "sub" else "sub",) + y[1:]
        return ANY

    def regs(s):  # scalar registers an operand names
        if s == "vcc":
            return {106, 107}
        m = re.match(r"s\[(\d+):(\d+)\]$|s(\d+)$", s)
        return set(range(int(m.group(1) or m.group(3)), int(m.group(2) or m.group(3)) + 1)) if m else set()

    def value(st, s):
        return ALL if s == "-1" else st.get(s, ANY)

    def assign(st, dst, v):
        if dst == "exec":
            st["exec"] = v
            return
        hit = regs(dst)
        for k in [k for k in st if k != "exec" and hit & regs(k)]:
            del st[k]
        if len(hit) == 2 and v != ANY:
            st[dst] = v

    def after(st, addr, op, a):
        if op.endswith("_saveexec_b64"):
            old, src = st["exec"], value(st, a[1])
            assign(st, a[0], old)
            if op.startswith("s_or_"):
                st["exec"] = either(old, src)
            elif op.startswith("s_andn2_"):  # src & ~exec
                st["exec"] = src if src[0] in ("sub", "diff") and either(src, old) == src[1] else ANY
            else:
                st["exec"] = ("sub", old, addr) if op.startswith("s_and_") else ANY
        elif op in ("s_or_b64", "s_xor_b64", "s_and_b64", "s_andn2_b64"):
            x, y = value(st, a[1]), value(st, a[2])
            v = ANY  # also the lanes a loop goes on with
            if op == "s_or_b64":
                v = either(x, y)
            elif op == "s_xor_b64":
                v = without(x, y) if without(x, y) != ANY else without(y, x)
            elif op == "s_and_b64" and a[0].startswith("s") and ALL in (x, y):
                v = ("sub", ALL, addr)
            assign(st, a[0], v)
        elif op == "s_mov_b64":
            assign(st, a[0], value(st, a[1]))
        elif a and re.match("[sv]_(?!cmp_.*_[iu]32$|cmp_.*_u64$|bitcmp)", op if op[0] == "s" else "v_"):
            for d in a[:2] if re.match("v_(div_scale|add_co|addc_co|sub_co|subb_co|mad_[ui]64)", op) else a[:1]:
                if d == "exec":
                    st["exec"] = ANY
                else:
                    assign(st, d, ANY)
            if op.startswith("v_cmpx"):
                st["exec"] = ANY

    seen, found = {}, set()
    work = [(0, (("exec", ALL),))]
    while work:
        i, key = work.pop()
        if key in seen.setdefault(i, set()):
            continue
        seen[i].add(key)
        assert len(seen[i]) <= 4096, "too many paths"
        st = dict(key)
        addr, op, args = ins[i]
        a = [x.strip() for x in args.split(",")] if args else []
        if op == "s_barrier" and st["exec"] != ALL:
            found.add(addr)
        nxt = [i + 1] if op not in ("s_branch", "s_endpgm") and i + 1 < len(ins) else []
        if op.startswith("s_cbranch") or op == "s_branch":
            off = int(a[0].split()[0])
            nxt.append(index[addr + 4 + 4 * (off - 65536 if off >= 32768 else off)])
        else:
            after(st, addr, op, a)
        if st["exec"] == ALL and op == "s_barrier":  # few masks live across one
            st = {r: v for r, v in st.items() if v == ALL}
        work += [(j, tuple(sorted(st.items()))) for j in nxt]
    return found


def test_barriers_are_reached_by_whole_waves(kernels):
    """The loops of the persistent kernels take their next item in one thread
    between barriers.  A compiler that sends the other lanes on to the barrier, or
    round the loop, without that thread leaves a barrier some lanes never reach."""
    names = [n for n in kernels if any(op == "s_barrier" for _, op, _ in kernels[n])]
    persistent = [n for n in names if "persistent" in n]
    assert len(persistent) >= 7
    for n in names:
        assert not exec_at_barriers(kernels[n]), n


def test_a_barrier_inside_a_divergent_branch_is_seen():
    """The shape that must not come out of the compiler: thread 0 reserves at the
    top of the loop, the other lanes pass it on their own and meet the barrier."""
    good = [(0, "v_cmp_eq_u32_e32", "vcc, 0, v0"), (4, "s_and_saveexec_b64", "s[2:3], vcc"),
            (8, "s_cbranch_execz", "1"), (12, "global_atomic_add", "v1, v2, v3, s[4:5] sc0"),
            (16, "s_or_b64", "exec, exec, s[2:3]"), (20, "s_barrier", ""), (24, "s_cbranch_scc1", "65529"),
            (28, "s_endpgm", "")]
    assert not exec_at_barriers(good)
    bad = [(0, "v_cmp_ne_u32_e32", "vcc, 0, v0"), (4, "s_and_saveexec_b64", "s[2:3], vcc"), (8, "s_barrier", ""),
           (12, "s_cbranch_scc1", "65534"), (16, "s_or_b64", "exec, exec, s[2:3]"), (20, "s_endpgm", "")]
    assert exec_at_barriers(bad) == {8}
