"""Loads written in inline asm have to wait for their data inside the same statement: the compiler takes the output
registers as written once the statement is over and may move, spill or reuse them while the load is still in flight.
(Loads that go to LDS have no output register.)"""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2206_07882_amd", "csrc")
LOAD = re.compile(r"\b(?:global_load|buffer_load|flat_load|scratch_load|s_load|ds_read|ds_load)_(?!lds)\w+")


def _unwaited(text):
    # runs of string literals (what a macro puts between them included): a statement's code
    runs = re.findall(r'"(?:[^"\\\n]|\\.)*"(?:[^;"{}()\n]*\\?\n?\s*"(?:[^"\\\n]|\\.)*")*', text)
    return [LOAD.search(r).group(0) for r in runs if LOAD.search(r) and "s_waitcnt" not in r]


def test_asm_loads_wait_in_their_own_statement():
    files = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")))
    assert len(files) > 10
    found = {os.path.basename(f): _unwaited(open(f).read()) for f in files}
    assert not any(found.values()), {k: v for k, v in found.items() if v}


def test_the_search_finds_what_it_looks_for():
    assert _unwaited('asm volatile("global_load_dwordx4 %0, %1, off" : "=&v"(v) : "v"(p));') == ["global_load_dwordx4"]
    assert _unwaited('#define LD(i) "buffer_load_dword %[v" #i "], %[o], %[r], 0 offen"') == ["buffer_load_dword"]
    assert not _unwaited('asm volatile("global_load_dword %0, %1, off\\n\\ts_waitcnt vmcnt(0)" : "=&v"(v) : "v"(p));')
    assert not _unwaited('asm volatile("global_load_lds_dwordx4 %0, off" ::"v"(p));')


WORD_USES = (r"qr_send\(word_at\(", r"\(void \*\)word_at\(",                # a store; where loads start
             r"__device__ __forceinline__ unsigned long long \*word_at\(int q, int hyp, int token\) const",
             r"auto word_at = \[&\]\(int q, int hyp, int token\) \{ return share\.word_at\(q, hyp, token\); \};")


def _other_word_uses(text):
    """Lines that mention a word's place (word_at, however it is written) or the area of the words itself, and are none of the above."""
    for use in WORD_USES:
        text = re.sub(use, "", text)
    return [line for line in text.splitlines() if re.search(r"\bword_at\b|\ba\.words\b", line) and "return a.words + b * a.n_words" not in line]


def test_words_between_workgroups_are_stored_by_their_helper_only():
    """A word of value and number that another workgroup polls has to be stored in one piece: by qr_send, never by an
    assignment that the compiler may split."""
    found = {}
    for f in glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")):
        text = open(f).read()
        if f.endswith("joint.hip"):
            assert len(re.findall(r"qr_send\(word_at\(", text)) >= 4
        found[os.path.basename(f)] = _other_word_uses(text)
    assert not any(found.values()), {k: v for k, v in found.items() if v}


def test_the_search_for_words_finds_other_uses():
    for line in ("*word_at(0, 1, 2) = v;", "(share.word_at)(q, 0, 0)[1] = v;", "auto *p = share.word_at(0, 0, 0);",
                 "unsigned long long *(word_at)(int q, int hyp, int token) const", "a.words[3] = 0;"):
        assert _other_word_uses(line) == [line]
    assert not _other_word_uses("qr_send(word_at(part, col, 4 * grp), sum, a.round);")
