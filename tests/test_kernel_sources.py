"""What has to hold in the text of the kernels because a run that broke it could touch memory that is not theirs."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_22175_amd", "csrc")


def _calls(text, name):
    """Argument lists of the calls of builtins whose name starts with `name`."""
    for m in re.finditer(re.escape(name) + r"\w*\(", text):
        depth, args, at = 1, [""], m.end()
        while depth:
            ch = text[at]
            depth += (ch in "([{") - (ch in ")]}")
            if ch == "," and depth == 1:
                args.append("")
            elif depth:
                args[-1] += ch
            at += 1
        yield [a.strip() for a in args]


def test_buffer_accesses_have_no_scalar_offset():
    """The scalar offset of a raw buffer access is no part of its bounds check; the epilogues rely on the check
    for rows past an expert's last, so every offset has to travel in the vector offset."""
    seen = 0
    for f in sorted(os.listdir(CSRC)):
        text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, f)).read())
        for kind, soffset in (("load", 2), ("store", 3)):
            for args in _calls(text, "__builtin_amdgcn_raw_buffer_" + kind):
                assert args[soffset] == "0", (f, args)
                seen += 1
    assert seen >= 15


def test_gate_weight_gradient_reads_the_expert_blocks_that_its_plan_has_room_for():
    """The plan sizes dL^T for EB blocks of sixteen experts and the kernel reads all blocks of its template argument, also
    those whose results it does not store: for each of the 64 numbers of experts the two have to be the same."""
    text = re.sub(r"//[^\n]*", "", open(os.path.join(CSRC, "permute.hip")).read())
    assert re.search(r"g\.EB = \(d\.E \+ 15\) / 16;", text) and "g.EB * 32 * g.tp_pad" in text
    launched = {int(blocks): int(kernel) for blocks, kernel in
                re.findall(r"(?:g\.EB == |case )(\d+)(?:\)|:) LAUNCH_DWG\((\d+)\);", text)}
    for E in range(1, 65):
        blocks = (E + 15) // 16
        assert launched.get(blocks) == blocks, E
