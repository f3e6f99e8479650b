"""The page kernels' item records (host code), and rounds whose sessions' agents do not have consecutive ids (GPU)."""
import dataclasses
import os
import subprocess

import numpy as np
import pytest

from paper_2604_03143_amd import workload as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_item_records(tmp_path):
    exe = str(tmp_path / "item_check")
    csrc = os.path.join(ROOT, "paper_2604_03143_amd", "csrc")
    cmd = ["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", csrc,
           os.path.join(ROOT, "tests", "item_check.cpp"), os.path.join(csrc, "tdk_plan.cpp"), "-o", exe]
    subprocess.run(cmd, check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr


def mixed(rnd, seed):
    """The same round with its agents listed in another order."""
    p = np.random.default_rng(seed).permutation(rnd.n_agents)
    return dataclasses.replace(rnd, agent_session=rnd.agent_session[p], agent_pos0=rnd.agent_pos0[p],
                               block_tables=[rnd.block_tables[i] for i in p], perturbed=[rnd.perturbed[i] for i in p],
                               segments=None if rnd.segments is None else [rnd.segments[i] for i in p])


@pytest.mark.gpu
@pytest.mark.parametrize("group,flags", [(0, None), (9, None), (32, None), (32, 191 + 512)])
@pytest.mark.parametrize("T,H", [(16, 8), (32, 2)])
def test_agents_listed_in_any_order(tdo, T, H, group, flags):
    """Groups of 1 to 21 agents (tables of up to 8, 16 and more agents are staged differently), ids in no order."""
    from test_gpu_parity import run_pipeline
    from test_gpu_ragged import ragged_round
    run_pipeline(tdo, mixed(ragged_round(T=T, H=H, spans=[333, 40, 100], agents=[21, 2, 10], stream=91), 3), group=group, flags=flags)


@pytest.mark.gpu
@pytest.mark.parametrize("group", [0, 32])
def test_agents_listed_in_any_order_with_own_block_orders(tdo, group):
    from test_gpu_parity import run_pipeline
    spec = wl.RoundSpec("mixed_perm", 92, 1, 4, 128, 16, 1.0e6, 2, 19, 5, 70, 3, 900, 0.2)
    rnd = wl.permute_blocks(wl.make_round(spec, spans=[350, 350], agents=[19, 6]), seed_tag=5)
    run_pipeline(tdo, mixed(rnd, 4), group=group)


@pytest.mark.gpu
def test_check_layer_with_agents_listed_in_any_order(tdo):
    from test_gpu_check_layer import run_case
    from test_gpu_ragged import ragged_round
    run_case(tdo, mixed(ragged_round(spans=[333, 40, 100], agents=[21, 2, 10], stream=93), 6), 0.15, 0.0, noise_everywhere=0.02)
