"""A shared word that one thread clears and others set needs a barrier between
the two: without one a late clear takes back a set that came before it.

This reads the kernels' sources: in every kernel, the first store to
a scalar `__shared__ int` by one thread and the next store to it by others have
a barrier between them."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2506_09463_amd", "csrc")
ONE = re.compile(r"if \((?:p\.pass == 1 && )?(?:tid|threadIdx\.x) == 0[^{;]*$")


def _kernels(text):
    """(name, body) of every __global__ function."""
    for m in re.finditer(r"__global__ void __launch_bounds__\([^)]*\)+\s*(\w+)\(", text):
        i = text.index("{", m.end())
        depth, j = 0, i
        while True:
            depth += {"{": 1, "}": -1}.get(text[j], 0)
            if depth == 0:
                break
            j += 1
        yield m.group(1), re.sub(r"//[^\n]*", "", text[i:j + 1])


def _one_thread(body, pos):
    """Whether the statement at pos is guarded by `if (tid == 0 ..)`, directly or
    by one of its enclosing blocks."""
    head = body[:pos].rstrip()
    start = max(head.rfind(c) for c in ";{}") + 1
    if ONE.search(head[start:].strip()):
        return True
    depth = 0
    for j in range(len(head) - 1, -1, -1):
        if head[j] == "}":
            depth += 1
        elif head[j] == "{":
            depth -= 1
            if depth < 0:
                depth = 0
                h = head[:j].rstrip()
                if ONE.search(h[max(h.rfind(c) for c in ";{}") + 1:].strip()):
                    return True
    return False


def unordered_flags(text):
    """(kernel, word) of every shared int whose clear by one thread and next
    store by others have no barrier between them."""
    bad = []
    for name, body in _kernels(text):
        for decl in re.findall(r"__shared__ int ([\w, ]+);", body):
            for word in decl.replace(" ", "").split(","):
                init = None
                for s in re.finditer(r"(?<![\w.>*])%s\s*=(?!=)" % word, body):
                    if _one_thread(body, s.start()):
                        init = s.end()
                    elif init is not None:
                        if "__syncthreads" not in body[init:s.start()]:
                            bad.append((name, word))
                        init = None
    return bad


def test_the_check_finds_an_unordered_flag():
    k = """__global__ void __launch_bounds__(64) k(int *p) {
    __shared__ int far, other;
    if (tid == 0) { far = 0; other = 0; }
    %s
    { int f = p[tid]; if (f) far = 1; }
    }"""
    assert unordered_flags(k % "") == [("k", "far")]
    assert unordered_flags(k % "__syncthreads();") == []


def test_shared_flags_are_ordered():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hpp"))):
        text = open(path).read()
        seen += len(list(_kernels(text)))
        assert unordered_flags(text) == [], os.path.basename(path)
    assert seen >= 30
