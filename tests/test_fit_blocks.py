"""The inline assembly of the fit's solver reads registers across lanes, and such a read needs two wait states after the vector
instruction that wrote the register.  The compiler does not look inside a block, nor does it know what a block begins with, so every
block has to see to that itself: for what it has written, and for what anything may have written just in front of it."""
import os
import re
import subprocess

SOURCE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2008_12260_amd", "csrc", "pollux_theta.hip")


def blocks():
    """The instructions of every asm statement, macros expanded."""
    text = "".join(ln for ln in open(SOURCE) if not ln.startswith("#include"))
    text = subprocess.run(["g++", "-E", "-P", "-x", "c++", "-"], input=text, check=True, capture_output=True, text=True).stdout
    for start in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
        pieces = re.match(r'(?:\s*"((?:[^"\\]|\\.)*)")+', text[start.end():])
        code = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', pieces.group(0)))
        instructions = [ln.strip() for ln in code.encode().decode("unicode_escape").splitlines() if ln.strip()]
        if instructions:
            yield instructions


def test_reads_across_lanes_wait_for_what_they_read():
    seen = 0
    for instructions in blocks():
        written, clock = {}, 0                                     # wait states since the block began, and at each register's write
        for ins in instructions:
            name, _, rest = ins.partition(" ")
            if name == "s_nop":
                clock += int(rest) + 1
                continue
            operands = [o.strip().lstrip("-").split(" ")[0] for o in rest.split(",")]
            if name.endswith("_dpp"):
                assert clock - written.get(operands[1], 0) >= 2, (ins, instructions)
                seen += 1
            clock += 1
            written[operands[0]] = clock
    assert seen >= 27 + 21                                         # the eliminations, the substitution
