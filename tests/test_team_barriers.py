"""What the compiler makes of the search kernels, looked at in its listing.

The wavefronts of a team exchange ids and counts through LDS: no barrier is reached while an LDS write is under way (a uint8 and a float row
variant stand for all; the code around the barriers is the same).  And a search with a key table takes no more vector registers
than one that gathers: with more, fewer wavefronts of a SIMD hide what they wait for."""
import os
import re
import subprocess

import pytest

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


def listing_of(source, directory):
    from paper_2512_02278_amd import build

    out = directory / "kernels.s"
    flags = [f for f in build.FLAGS if not f.startswith("-Rpass")]
    subprocess.run(["hipcc", *flags, "--offload-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
    return out.read_text()


def check_barriers(listing):
    kernels = [(name, body) for name, body in functions(listing) if any(op == "s_barrier" for op, _ in body)]
    teams = [name for name, _ in kernels if re.search(r"Li[24]ELb0E", name)]
    assert len(teams) == 14  # seven list variants, two and four wavefronts
    assert not [name for name, body in kernels if barriers_reached_with_writes_under_way(body)]


def test_team_kernels_wait_for_their_lds_writes_before_barriers(tmp_path):
    check_barriers(listing_of("inst_u8_l2_g8n1.hip", tmp_path))


@pytest.fixture(scope="module")
def float_listing(tmp_path_factory):
    return listing_of("inst_f32_l2_g8n3.hip", tmp_path_factory.mktemp("listing"))


def test_team_kernels_over_float_rows_wait_for_their_lds_writes_before_barriers(float_listing):
    check_barriers(float_listing)


def test_search_with_a_key_table_takes_no_more_registers_than_gathering(float_listing):
    registers = {}
    for entry in re.findall(r"- \.agpr_count.*?\.wavefront_size", float_listing, re.S):
        name = re.search(r"\.name:\s+(\S+)", entry).group(1)
        registers[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", entry).group(1))
    table = {n: v for n, v in registers.items() if re.search(r"18beam_search_kernel.*Li1ELb1E", n)}
    assert len(table) == 7
    for name, count in table.items():
        assert count <= registers[name.replace("Li1ELb1E", "Li1ELb0E")], name
