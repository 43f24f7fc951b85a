"""The copy threads of a swapping volume, on the CPU: the pool's header is
built with g++ into a small program for each case (it uses no HIP)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1708_00783_amd", "csrc")

HEAD = r"""
#include "tsdf_copy_pool.h"
#include <signal.h>
#include <stdlib.h>
#include <stdio.h>
#include <sys/resource.h>
#include <sys/wait.h>
#include <time.h>
using tsdf::CopyPool;
struct Count : CopyPool::Job {
    uint32_t n;
    std::vector<std::atomic<uint32_t>> hits;
    explicit Count(uint32_t blocks) : n(blocks), hits(blocks) {}
    uint32_t size() const override { return n; }
    void block(uint32_t k) override { hits[k].fetch_add(1); }
    bool whole() const
    {
        for (const auto &h : hits)
            if (h.load() != 1) return false;
        return true;
    }
};
static bool copy_all(CopyPool &pool, uint32_t n)
{
    Count job(n);
    job.per = (n + CopyPool::kParts - 1) / CopyPool::kParts;
    pool.start(job);
    for (uint32_t p = 0, at = 0; at < n; ++p, at += job.per)
        CopyPool::finish_part(job, p, n - at < job.per ? n - at : job.per);
    pool.finish();
    return job.whole();
}
"""


def run(tmp_path, body, args=(), timeout=60):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(HEAD + body)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-pthread", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    return subprocess.run([str(exe), *map(str, args)], timeout=timeout, capture_output=True, text=True)


@pytest.mark.parametrize("blocks", [1, 15, 16, 17, 128, 1000, 4097])
def test_every_block_is_copied_once(tmp_path, blocks):
    r = run(tmp_path, r"""
int main(int, char **a)
{
    CopyPool pool;
    for (int k = 0; k < 200; ++k)
        if (!copy_all(pool, (uint32_t)atoi(a[1]))) return 1;
    return 0;
}
""", [blocks])
    assert r.returncode == 0, r.stderr


def test_a_forked_child_ends_with_the_pool(tmp_path):
    """The child destroys its copy of a pool whose helpers, asleep, exist in
    the parent alone; the parent's goes on working and ends too."""
    r = run(tmp_path, r"""
int main()
{
    CopyPool *pool = new CopyPool();
    if (!copy_all(*pool, 500)) return 1;
    usleep(100000);                       // the helpers are asleep again
    const pid_t child = fork();
    if (child == 0) {
        delete pool;
        _exit(0);
    }
    int st = -1;
    for (int k = 0; k < 100; ++k, usleep(100000))
        if (waitpid(child, &st, WNOHANG) == child) break;
    if (st != 0) {
        kill(child, SIGKILL);
        waitpid(child, &st, 0);
        fprintf(stderr, "the child hangs\n");
        return 2;
    }
    const bool ok = copy_all(*pool, 500);
    delete pool;
    return ok ? 0 : 3;
}
""")
    assert r.returncode == 0, r.stderr


def test_helpers_sleep_when_a_job_has_no_more_blocks(tmp_path):
    """Between the last block taken and finish() -- a wait for the device -- the helpers use no CPU time."""
    r = run(tmp_path, r"""
int main()
{
    CopyPool pool;
    if (!copy_all(pool, 500)) return 1;
    Count job(500);
    pool.start(job);
    CopyPool::finish_part(job, 0, 500);
    struct rusage a, b;
    getrusage(RUSAGE_SELF, &a);
    usleep(400000);
    getrusage(RUSAGE_SELF, &b);
    pool.finish();
    const double used = (b.ru_utime.tv_sec - a.ru_utime.tv_sec) + 1e-6 * (b.ru_utime.tv_usec - a.ru_utime.tv_usec);
    printf("%.3f s\n", used);
    return job.whole() && used < 0.1 ? 0 : 2;
}
""")
    assert r.returncode == 0, r.stdout


def test_a_wait_for_a_block_gives_up_its_core(tmp_path):
    """Blocks that come late are waited for asleep, not spinning."""
    r = run(tmp_path, r"""
struct Late : Count {
    std::atomic<bool> there{false};
    using Count::Count;
    void block(uint32_t k) override
    {
        for (CopyPool::Turn turn; !there.load();) turn();
        Count::block(k);
    }
};
int main()
{
    CopyPool pool;
    if (!copy_all(pool, 500)) return 1;
    Late job(500);
    pool.start(job);
    struct rusage a, b;
    getrusage(RUSAGE_SELF, &a);
    usleep(400000);
    getrusage(RUSAGE_SELF, &b);
    job.there = true;
    CopyPool::finish_part(job, 0, 500);
    pool.finish();
    const double used = (b.ru_utime.tv_sec - a.ru_utime.tv_sec) + 1e-6 * (b.ru_utime.tv_usec - a.ru_utime.tv_usec);
    printf("%.3f s\n", used);
    return job.whole() && used < 0.3 ? 0 : 2;
}
""")
    assert r.returncode == 0, r.stdout
