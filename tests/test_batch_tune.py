"""The autotuned choices of a batched solve hold for the class of batch that
they were timed on (CPU: the library's rules in a program of their own)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1008_1371_amd", "csrc")

PROGRAM = r"""
#include "batch_tune.h"
// arguments: cache text, then queries "problems nmax mixed" on 256 compute units
int main(int argc, char **argv)
{
    hsvd::BatchTune t;
    t.read(argv[1]);
    bool first = true;
    for (int k = 2; k < argc; ++k) {
        int problems, nmax, mixed;
        if (sscanf(argv[k], "%d %d %d", &problems, &nmax, &mixed) != 3) return 1;
        printf("%d %d\n", t.threads_for(problems, nmax, 256), t.schedule_for(problems, nmax, 256, mixed != 0));
    }
    printf("%d %d\n", t.last[0], t.last[1]);
    t.write(stdout, first);
    return 0;
}
"""


@pytest.fixture(scope="module")
def choices(tmp_path_factory):
    d = tmp_path_factory.mktemp("batch_tune")
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(d / "main.cpp"), "-o", str(d / "main")],
                   check=True, timeout=120)

    def run(cache, *queries):
        r = subprocess.run([str(d / "main"), cache, *queries], capture_output=True, text=True, check=True, timeout=20)
        lines = r.stdout.split("\n")
        k = len(queries)
        return ([tuple(map(int, line.split())) for line in lines[:k]], tuple(map(int, lines[k].split())),
                "\n".join(lines[k + 1:]))
    return run


ALL = ["16 256 0", "300 256 0", "500 256 0", "1500 256 0", "4000 256 0", "4000 64 0", "16 256 1"]
UNTUNED = [(1024, 1), (1024, 1), (1024, 0), (512, 0), (256, 0), (256, 0), (1024, 0)]


def test_untuned(choices):
    assert choices("", *ALL) == (UNTUNED, (-1, -1), "")


def test_a_large_batch_does_not_decide_for_a_small_one(choices):
    """Tuned on thousands of problems: the persistent launch, 256 threads.
    Batches of fewer problems keep the rule's choice."""
    cache = ('{"entries": [{"batched_bucket": 3, "threads": 256, "problems_class": 4}, '
             '{"batched_schedule": 0, "mode": 0, "problems_class": 4}]}')
    assert choices(cache, *ALL)[0] == UNTUNED


def test_nor_a_small_batch_for_a_large_one(choices):
    cache = ('{"batched_bucket": 3, "threads": 512, "problems_class": 0}, '
             '{"batched_schedule": 0, "mode": 1, "problems_class": 0}, '
             '{"batched_schedule": 1, "mode": 1, "problems_class": 0}')
    got, last, text = choices(cache, *ALL)
    assert got == [(512, 1)] + UNTUNED[1:6] + [(512, 1)]
    assert last == (1, 1)
    assert choices(text, *ALL) == (got, last, text)  # what is written is what is read


@pytest.mark.parametrize("problems,count_class", [(1, 0), (128, 0), (129, 1), (320, 1), (321, 2), (768, 2), (769, 3),
                                                  (1792, 3), (1793, 4), (100000, 4)])
def test_classes_end_at_the_lines_of_the_rules(choices, problems, count_class):
    for c in range(5):
        cache = '{"batched_bucket": 0, "threads": 1024, "problems_class": %d}' % c
        assert (choices(cache, "%d 64 0" % problems)[0][0][0] == 1024) == (c == count_class)


def test_entries_without_a_class_hold_for_all(choices):
    """Files of former versions."""
    cache = '{"batched_bucket": 3, "threads": 512},\n {"batched_schedule": 0, "mode": 1}\n'
    got, last, _ = choices(cache, *ALL)
    assert got == [(512, 1)] * 5 + [(256, 1), (512, 0)]
    assert last == (1, -1)


@pytest.mark.parametrize("entry", ['"batched_bucket": 4, "threads": 256', '"batched_bucket": 3, "threads": 128',
                                   '"batched_bucket": 3, "threads": 256, "problems_class": 5',
                                   '"batched_bucket": 3, "threads": 256, "problems_class": -1',
                                   '"batched_schedule": 2, "mode": 1', '"batched_schedule": 0, "mode": 2',
                                   '"batched_schedule": 0, "mode": 0, "problems_class": 9'])
def test_bad_entries_are_ignored(choices, entry):
    assert choices("{%s}" % entry, *ALL)[0] == UNTUNED
