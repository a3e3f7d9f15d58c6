"""Row blocks cut where a workgroup slot is full: splits of unequal length.

CPU: tests/work_split.cpp checks that the work lists of random ragged batches cover
every key tile of every row block exactly once.  GPU: few compute units are declared, so
that small batches are cut this way, for row blocks of each size and each key source."""
import os
import shutil
import subprocess

import pytest
import torch  # noqa: F401  (before the library, so that both share one HIP runtime)

import paper_2607_17715_amd as c2kv
import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is not installed")
def test_work_list_covers_every_tile_once(tmp_path):
    exe = str(tmp_path / "work_split")
    csrc = os.path.join(ROOT, "paper_2607_17715_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "work_split.cpp"),
                    os.path.join(csrc, "plan.cpp"), "-o", exe], check=True, timeout=300)
    r = subprocess.run([exe, "400", "3"], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:]
    assert int(r.stdout.split()[3]) > 40, r.stdout


CASES = [
    # 64-row blocks, paged and pool: one row block per (request, kv-head)
    (dict(batch=5, n_q_heads=8, n_kv_heads=4, suffix_len=2, chunks_per_req=4, chunk_len=400), 8),
    # 128-row blocks, int8
    (dict(batch=5, n_q_heads=8, n_kv_heads=2, suffix_len=29, chunks_per_req=4, chunk_len=400,
          pool_dtype="i8"), 8),
    # 256-row blocks, the last of a request short, head_dim 64
    (dict(batch=5, n_q_heads=12, n_kv_heads=4, suffix_len=101, chunks_per_req=4, chunk_len=500,
          head_dim=64), 32),
    # fp32
    (dict(batch=3, n_q_heads=4, n_kv_heads=4, suffix_len=70, chunks_per_req=4, chunk_len=500,
          pool_dtype="f32"), 24),
]


def test_one_round_of_even_splits_is_kept():
    """24 fp32 row blocks of 256 rows, 5 to 17 tiles each: pieces of one and two tiles fit one
    round of 256 slots, so they are not cut into fewer and longer ones."""
    w = synth.small(pool_dtype="f32", n_q_heads=8, n_kv_heads=2, batch=1, chunks_per_req=2,
                    keep=("count", 130), prefix_len=0, suffix_len=744, seed=3)
    i = c2kv.Plan.for_workload(w).info
    assert i["rows_per_block"] == 256 and i["n_merge_groups"] == 24
    assert 200 < i["n_work_items"] <= 256, i


@pytest.mark.gpu
@pytest.mark.parametrize("shape,num_cus", CASES)
def test_cut_row_blocks_parity(shape, num_cus):
    from test_gpu_parity import _both_paths
    w = synth.small(seed=31, keep=("ratio", 0.4, 0.9), **shape)
    plan = _both_paths(w, f"cut {shape}", num_cus=num_cus)
    i = plan.info
    groups = w.batch * w.n_kv_heads * -(-w.suffix_len * (w.n_q_heads // w.n_kv_heads) //
                                        i["rows_per_block"])
    assert i["n_merge_groups"] > 0 and i["n_work_items"] % groups != 0, (groups, i)
