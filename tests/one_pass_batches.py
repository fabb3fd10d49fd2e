"""Batches whose backward the planner runs in one pass, with the sizes at which that can go wrong among their documents."""
import random

from paper_2510_18121_amd import workloads as W


def _documents(lens, shard, hq, hkv, d, extra_keys=0, gap=0):
    """Ragged documents in shuffled shards; `extra_keys` behind each document's last query; every `gap`-th shard is not in the batch."""
    tasks = [(i, a, min(shard, n - a)) for i, n in enumerate(lens) for a in range(0, n, shard)]
    if gap:
        tasks = [t for k, t in enumerate(tasks) if k % gap]
    random.Random(len(lens)).shuffle(tasks)
    return W.custom([n + extra_keys for n in lens], tasks, hq, hkv, d, task_order=list(range(len(tasks))))


# one row, packed blocks of 16 and 32 rows, edges of steps (32), blocks (64) and key tiles (128, 256)
EDGES = [1, 5, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513]

BATCHES = {
    "documents": lambda: _documents([8001, 7000, 6001, 5000, 4001, 3000] + EDGES, 300, 32, 8, 128),
    "gaps_and_keys_nobody_sees": lambda: _documents([6001, 6000] * 3 + EDGES, 77, 16, 8, 128, extra_keys=301, gap=7),
    "windows": lambda: W.split_kv(W.custom([60001, 700, 33], [(0, 59338, 663), (1, 0, 700), (2, 0, 33)], 32, 8, 128), 2253)[0],
    "shards_d64": lambda: W.custom([90001, 89000] + EDGES, [(0, 87829, 2172), (1, 86828, 2172)] + [(2 + i, 0, n) for i, n in enumerate(EDGES)], 32, 8, 64),
    # where moving K and V costs the other kernels much, and a short list at head_dim 64
    "short_shards": lambda: W.shard_chunk(61, "distinct", seed=3, chunk_tokens=61 * 140, max_context=3000, hq=16, hkv=16, d=128),
    "short_documents_d64": lambda: _documents([4001, 3000, 2049, 2048, 2047, 1900, 1500, 1024] + EDGES, 0x7fffffff, 16, 16, 64),
    # sums of dQ just within 4 GiB: the largest 32-bit offsets
    "offsets_up_to_4_gib": lambda: _documents([1023] * 127 + [959], 300, 64, 8, 128),
    "documents_d64": lambda: _documents([8001, 8000] * 3 + EDGES, 1029, 16, 16, 64),
}
