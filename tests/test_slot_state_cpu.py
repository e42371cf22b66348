"""Of the slots of time of an env only slot 0 reads its state: the others draw theirs, and slot 0 may have written it by then.
Checked in the sources: in every kernel that has an instance for slots a read of the state stands under a test of `head`."""
import glob
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2311_10090_amd", "csrc")
READ = re.compile(r"(?:[\w.\[\]]+\s*=[^=;]*?\bA\.st\.(?:pos_a|vel_a|pos_l)\s*\[|\bload_state<)")


def slot_kernels():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        for m in re.finditer(r"__global__[^;{]*?\b(\w+_kernel)\(", text):
            start = text.index("{", m.end())
            depth, end = 1, start + 1
            while depth:
                depth += {"{": 1, "}": -1}.get(text[end], 0)
                end += 1
            body = text[start:end]
            if re.search(r"kSlots<|\bSLOTS\b", body):
                yield m[1], body


def unguarded_reads(body):
    """Statements that read the state under no condition with `head`: of the blocks around them, or of their own."""
    out, stack, closed, begin = [], [], "", 0
    for k, c in enumerate(body):
        if c not in "{};":
            continue
        head = body[begin:k].strip()
        if c == "{":
            if head.startswith("else"):
                head = closed + " " + head                   # an else branch has its if's condition too
            stack.append(head)
        else:
            if READ.search(head) and not any(re.search(r"\bhead\b", s) for s in stack + [head]):
                out.append(head)
            closed = stack.pop() if c == "}" and stack else ("" if not head.startswith("if") else head)
        begin = k + 1
    return out


def test_reads_are_found():
    assert unguarded_reads("{ if (valid) { px = A.st.pos_a[g]; } }") and unguarded_reads("{ if (valid) load_state<N>(s, A.st, TE, g); }")
    assert unguarded_reads("{ if (head) { } lx = ok ? A.st.pos_l[g] : 0.0f; }")
    assert not unguarded_reads("{ if (valid && head) { px = A.st.pos_a[g]; } else if (ok) { vx = A.st.vel_a[g]; } }")
    assert not unguarded_reads("{ if (valid) { A.st.pos_a[g] = px; } if (head) load_state<N>(s, A.st, TE, g); ep = A.st.ep_step[g]; }")


KERNELS = list(slot_kernels())


def test_every_kernel_is_seen():
    assert {name for name, _ in KERNELS} == {"rollout_agents_kernel", "rollout_uniform_ws_kernel", "rollout_small_kernel", "rollout_waves_kernel",
                                             "rollout_gru_kernel", "rollout_gru_waves_kernel"}


@pytest.mark.parametrize("name,body", KERNELS, ids=[name for name, _ in KERNELS])
def test_only_slot_0_reads_the_state(name, body):
    assert READ.search(body) and unguarded_reads(body) == []
