"""LDS rings, looked at in the assembly: what a barrier hands on, and which rows a
stage's loads may reach.

No wave may pass a barrier with reads of the stage before in flight.

The staged kernels hand a ring's stage on at a barrier: behind it the waves
refill the stage that the previous step read.  A read that a wave has issued but
not waited for would then race with the refill, and no run can be relied on to
show it.  So the assembly is looked at: along every path, the LDS reads that may
be outstanding at each s_barrier.
"""

import os
import re
import subprocess

import pytest

from paper_2609_36899_amd import build

SOURCES = ["gemm.hip", "attention_prefill.hip"]


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    """Kernel name -> instruction lines, for the sources with LDS rings."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    out = tmp_path_factory.mktemp("asm")
    procs = [subprocess.Popen([build.HIPCC, *build.HIP_FLAGS, "-x", "hip", "--cuda-device-only", "-S",
                               os.path.join(build.CSRC, s), "-o", str(out / s)],
                              stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)
             for s in SOURCES]
    assert [p.wait() for p in procs] == [0] * len(SOURCES)
    return {m[1]: m[2] for s in SOURCES for m in
            re.finditer(r"^(\w+):\s*; @\1\n(.*?)^\.Lfunc_end", (out / s).read_text(), re.M | re.S)}


def _blocks(body):
    """[(label, instructions)] in program order."""
    blocks = [("entry", [])]
    for line in body.splitlines():
        line = line.split(";")[0].strip()
        label = re.match(r"(\.LBB\w+):", line)
        if label:
            blocks.append((label[1], []))
        elif line and not line.startswith("."):
            blocks[-1][1].append(line)
    return blocks


def reads_at_barriers(body):
    """The largest number of LDS reads in flight at each s_barrier (LDS operations
    of a wave complete in order, so a wait for n leaves at most n)."""
    blocks = _blocks(body)
    at = {label: i for i, (label, _) in enumerate(blocks)}
    entry, found, todo = {0: 0}, {}, [0]

    def flow(i, n):
        if i < len(blocks) and n > entry.get(i, -1):
            entry[i] = n
            todo.append(i)

    while todo:
        i = todo.pop()
        n, code = entry[i], blocks[i][1]
        for k, ins in enumerate(code):
            op = ins.split()[0]
            if op.startswith("ds_read"):
                n += 1
            elif op == "s_waitcnt":
                wait = re.search(r"lgkmcnt\((\d+)\)", ins)
                n = min(n, int(wait[1])) if wait else n
            elif op == "s_barrier":
                found[i, k] = n
            elif op == "s_branch":
                flow(at[ins.split()[1]], n)
                break
            elif op.startswith("s_cbranch"):
                # "no lane active" ahead of a jump to the other arm of a uniform
                # branch: not taken, a wave arrives here with lanes active.
                if op == "s_cbranch_execz" and code[k + 1:k + 2] and \
                        code[k + 1].split()[0] == "s_branch":
                    continue
                flow(at[ins.split()[1]], n)
            elif op == "s_endpgm":
                break
        else:
            flow(i + 1, n)
    return list(found.values())


def test_wait_counts_follow_every_path():
    loop = ("ds_read_b128 v[0:3], v9\n.LBB0_1:\ns_waitcnt lgkmcnt(%d)\ns_barrier\n"
            "ds_read_b128 v[0:3], v9\nds_read_b128 v[4:7], v9\ns_cbranch_scc1 .LBB0_1\ns_endpgm\n")
    assert reads_at_barriers(loop % 0) == [0]
    assert reads_at_barriers(loop % 1) == [1]  # of the two that the back edge brings


@pytest.mark.parametrize("kernel", ["gemm_bf16_tileILi64E", "gemm_bf16_tileILi128E",
                                    "gemm_bf16_tileILi192E", "gemm_bf16_tileILi256E",
                                    "gemm_bf16_wide", "attn_prefill_bf16"])
def test_no_lds_read_in_flight_at_a_barrier(assembly, kernel):
    forms = {name: body for name, body in assembly.items() if kernel in name}
    assert len(forms) >= 2
    for name, body in forms.items():
        left = reads_at_barriers(body)
        assert left and max(left) == 0, (name, left)


@pytest.mark.parametrize("kernel", ["gemm_bf16_tile", "gemm_bf16_wide", "attn_prefill_bf16ILi128Et"])
def test_no_load_between_the_wait_and_its_barrier(assembly, kernel):
    """wait_vmem counts what was issued before it: a load into LDS that had moved
    behind it would pass the barrier uncounted."""
    for name, body in assembly.items():
        if kernel not in name:
            continue
        for _, code in _blocks(body):
            for k, ins in enumerate(code):
                if ins.startswith("s_barrier"):
                    back = code[:k][::-1]
                    wait = next(j for j, b in enumerate(back) if "vmcnt" in b)
                    assert not [b for b in back[:wait] if re.search(r"load_lds|\blds$", b)], name


def test_rows_past_the_batch_are_kept_out_by_the_lane_offset(assembly):
    """The last M-block of the 256 x 256 tile addresses rows past M.  Its buffer ends
    at row M, and the bounds check is certain only of the lane's offset, not of the
    uniform one: the eight loads of an A stage, 32 rows apart, must differ in the
    lane's offset and share the uniform one."""
    forms = [body for name, body in assembly.items() if "gemm_bf16_wide" in name]
    assert len(forms) == 2
    for body in forms:
        loads = re.findall(r"buffer_load_dwordx4 (v\d+), s\[[\d:]+\], (\w+) offen(.*)", body)
        a = [(lane, uniform) for lane, uniform, flags in loads if "nt" not in flags.split()]
        assert a and len(a) % 8 == 0
        for i in range(0, len(a), 8):
            assert len({lane for lane, _ in a[i:i + 8]}) == 8
            assert len({uniform for _, uniform in a[i:i + 8]}) == 1
