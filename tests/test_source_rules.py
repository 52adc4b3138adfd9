"""Rules that the kernels' sources keep, checked without a GPU."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1610_02132_amd", "csrc")


def body(text, at):
    """The {...} block that opens at or after `at`."""
    start = text.index("{", at)
    depth = 0
    for i in range(start, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[start:i + 1]
    raise AssertionError("no closing brace")


def kernels():
    """(file, name, wavefronts of a workgroup are more than one, body, text of the file)"""
    for name in sorted(os.listdir(CSRC)):
        if name.endswith(".hip"):
            text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, name)).read())
            for m in re.finditer(r"__global__(?P<attr>[^;{]*?)\bvoid\s+(?P<name>k_\w+)\(|"
                                 r"__global__\s+void\s+(?P<name2>k_\w+)\(", text):
                one = re.search(r"__launch_bounds__\(64\)", m.group("attr") or "")
                yield name, m.group("name") or m.group("name2"), not one, body(text, m.end()), text


def uses_barrier(block, text, depth=3):
    if "__syncthreads" in block:
        return True
    called = set(re.findall(r"\b([a-z_]\w+)\s*\(", block)) if depth else ()
    for f in called:
        d = re.search(r"__device__[^;{]*\b%s\([^;{]*\)\s*\{" % f, text)
        if d and uses_barrier(body(text, d.start()), text, depth - 1):
            return True
    return False


def test_wavefronts_of_a_workgroup_leave_together():
    """The status word is written by other workgroups of the same launch: where wavefronts meet at
    barriers, none of them may leave on its own reading of it."""
    seen = []
    for file, name, several, block, text in kernels():
        alone = re.search(r"if\s*\(\s*\*\s*a\.status\s*!=\s*0\s*\)\s*return", block)
        seen.append(name)
        if several and uses_barrier(block, text):
            assert not alone, f"{file}: {name} leaves wavefront by wavefront"
    for name in ("k_decode_split", "k_decode_tile", "k_sparse_resolve", "k_gen_parse_entries", "k_raw_apply"):
        assert name in seen


def test_loops_over_a_long_buckets_values_count_in_64_bits():
    """A bucket of the general path has up to 2^32 - 1 values: an index of 32 bits that a stride takes
    past such an end starts over, and the loop does not end."""
    text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "qsgd_general.hip")).read())
    loops = re.findall(r"for \((\w+) (\w+) = [^;]*threadIdx\.x[^;]*; \2 < (?:m|a\.n); \2 \+= ", text)
    assert len(loops) >= 3
    assert all(kind == "uint64_t" for kind, _ in loops), loops


def test_arrays_stored_16_bytes_at_a_time_say_so():
    """An array of words in LDS is aligned to 4 bytes unless it says otherwise."""
    seen = []
    for file, name, _, block, _ in kernels():
        for array in set(re.findall(r"reinterpret_cast<uint4\s*\*>\((\w+)\)\[", block)):
            decl = re.search(r"[^;{}]*__shared__[^;]*\b%s\[" % array, block)
            if decl:
                seen.append((file, array))
                assert "aligned(16)" in decl.group(0), f"{file}: {name}: {array}"
    assert len(seen) >= 2


def test_every_device_function_has_a_caller():
    text = "".join(re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, n)).read()) for n in sorted(os.listdir(CSRC)))
    names = set(re.findall(r"__device__\b[^;{}()]*?\b(\w+)\([^;{]*\)\s*\{", text))
    assert len(names) >= 40
    alone = [n for n in sorted(names) if len(re.findall(r"\b%s\b" % n, text)) < 2]
    assert not alone, alone
