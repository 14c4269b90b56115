"""The wavefronts of a team exchange ids and counts through LDS: no barrier of the search kernels is reached while an LDS write is under
way.  Looked at in the listing that the compiler makes of them (one row variant stands for all; the code around the barriers is
the same)."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def functions(listing):
    """(name, [(operation, operands) or ("label", name)]) of every kernel."""
    found, body = [], None
    for line in listing.split("\n"):
        m = re.match(r"(_Z\w+):", line)
        if m:
            body = []
            found.append((m.group(1), body))
        elif line.startswith(".Lfunc_end"):
            body = None
        elif body is not None:
            m = re.match(r"(\.LBB\w+):", line)
            if m:
                body.append(("label", m.group(1)))
                continue
            m = re.match(r"\s+([a-z]\w+)(.*)", line)
            if m:
                body.append((m.group(1), m.group(2).split(";")[0].strip()))
    return found


def barriers_reached_with_writes_under_way(body):
    """Along every path: an LDS write leaves one under way, a wait for all LDS operations none."""
    at = {operand: i for i, (op, operand) in enumerate(body) if op == "label"}
    after = {}
    for i, (op, operand) in enumerate(body):
        if op.startswith("s_cbranch") or op == "s_branch":
            after.setdefault(i, []).append(at[operand])
        if op not in ("s_branch", "s_endpgm", "s_setpc_b64") and i + 1 < len(body):
            after.setdefault(i, []).append(i + 1)
    under_way, todo = {0: False}, [0]
    while todo:
        i = todo.pop()
        op, operand = body[i]
        state = under_way[i]
        if op.startswith("ds_") and not op.startswith("ds_read") and "permute" not in op and "swizzle" not in op:
            state = True
        elif op == "s_waitcnt" and "lgkmcnt(0)" in operand:
            state = False
        for t in after.get(i, []):
            if t not in under_way or (state and not under_way[t]):
                under_way[t] = state or under_way.get(t, False)
                todo.append(t)
    return [i for i, (op, _) in enumerate(body) if op == "s_barrier" and under_way.get(i)]


def test_the_check_sees_a_missing_wait():
    loop = [("label", ".LBB0_1"), ("s_barrier", ""), ("ds_write_b32", "v0, v1"), ("s_cbranch_scc1", ".LBB0_1"), ("s_endpgm", "")]
    assert barriers_reached_with_writes_under_way(loop) == [1]
    loop.insert(3, ("s_waitcnt", "lgkmcnt(0)"))
    assert not barriers_reached_with_writes_under_way(loop)


def test_team_kernels_wait_for_their_lds_writes_before_barriers(tmp_path):
    from paper_2512_02278_amd import build

    out = tmp_path / "kernels.s"
    flags = [f for f in build.FLAGS if not f.startswith("-Rpass")]
    subprocess.run(["hipcc", *flags, "--offload-device-only", "-S", os.path.join(build.CSRC, "inst_u8_l2_g8n1.hip"), "-o", str(out)], check=True, capture_output=True)
    kernels = [(name, body) for name, body in functions(out.read_text()) if any(op == "s_barrier" for op, _ in body)]
    teams = [name for name, _ in kernels if re.search(r"Li[24]ELb0E", name)]
    assert len(teams) == 14  # seven list variants, two and four wavefronts
    assert not [name for name, body in kernels if barriers_reached_with_writes_under_way(body)]
