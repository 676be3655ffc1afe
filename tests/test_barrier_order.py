"""Where the kernels' barriers stand, read off the sources (no GPU needed): a word in LDS that one thread
rewrites is only rewritten after a barrier that every reader of its old value has passed.  A wavefront that
reads the new value takes another branch than the others, and the branches hold barriers of their own: the
workgroup falls out of step.  That cannot be shown by running it, so the order itself is checked."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_04541_amd", "csrc")


def source(name: str) -> str:
    text = open(os.path.join(CSRC, name)).read()
    return re.sub(r"//[^\n]*", "", re.sub(r"/\*.*?\*/", "", text, flags=re.S))


def block_after(text: str, head: str) -> str:
    """The braced block that follows the (only) occurrence of `head`, braces included."""
    assert text.count(head) == 1, head
    at = text.index("{", text.index(head) + len(head))
    depth = 0
    for i in range(at, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[at:i + 1]
    raise AssertionError("unbalanced braces after " + head)


def events(text: str, **patterns: str) -> list:
    """Names of the patterns in the order in which they occur; "barrier" is always among them."""
    patterns = dict(patterns, barrier=r"__syncthreads\(\)")
    joined = "|".join("(?P<%s>%s)" % kv for kv in patterns.items())
    return [m.lastgroup for m in re.finditer(joined, text)]


def test_the_place_of_a_piece_is_rewritten_between_barriers():
    kinds = block_after(source("lychee_layer.hip"), "for (int kind = 0; kind < 2; ++kind)")
    loop = block_after(kinds, "for (;;)")
    # where() reads the words of pool.run that thread 0 writes
    seen = events(kinds.replace("auto where = [&]", ""), read=r"\bwhere\(\);", write=r"pool\.run\[\d\] = ")
    assert seen.count("read") == 2 and seen.count("write") == 5, seen
    order = [e for i, e in enumerate(seen) if i == 0 or e != seen[i - 1]]  # (runs of one event are one)
    for a, b in zip(order, order[1:]):
        assert {a, b} != {"read", "write"}, "no barrier between a %s and the %s after it: %s" % (a, b, order)
    # the loop is left right after its first read, and the next kind's set-up writes
    after = kinds[kinds.index(loop) + len(loop):]
    assert events(after) == ["barrier"], "no barrier between the loop's last read and the next kind's set-up"


def test_the_count_of_the_last_entries_is_read_before_it_is_reset():
    rule = block_after(source("lychee_select.h"), "__device__ __forceinline__ int rule_keeps")
    read = r"uni\(sh\.n_last\)"
    assert len(re.findall(read, rule)) == 1
    # (right after the read, ahead of every branch: the ways out of the loop differ in what they do next)
    assert re.match(r";\s*__syncthreads\(\);", rule[re.search(read, rule).end():]), "no barrier right after the read"


def test_the_answer_of_the_list_reservation_is_waited_for_after_the_merge():
    """In a pooled piece the last wavefront asks for the room of the piece's last candidates and, of four heads, merges
    one: it stores the answer, which it waits for, behind that, and ahead of the barrier that the readers pass."""
    piece = block_after(source("lychee_stream.h"), "__device__ __forceinline__ void run_piece")
    seen = events(piece[piece.index("int cand_base = 0;"):], ask=r"cand_base = __hip_atomic_fetch_add", answer=r"sh\.cand_base = cand_base",
                  merge=r"if \(uni\(wave\) < NH\)", read=r"int base = sh\.cand_base")
    assert seen == ["ask", "barrier", "merge", "answer", "barrier", "read"], seen
