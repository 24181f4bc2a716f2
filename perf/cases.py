"""The workloads that this library's speed is judged by, through its Python entry points.

Every case is one call that a program makes once its key schedule, buffers,
message records or work list are in hand.  Sizes are the paper's file sizes
(1,202 ... 1,190,402 bytes, section 5), those of bench.py and of the tests, or
plain powers of two.  Outputs are cipher bytes, for which only one answer is
right, so they are compared for equality and no wider reference is given.
The serving engine runs the kernel of the `batch` cases.
"""
import functools

import numpy as np
import torch

from paper_1902_05234_amd import aes, batch, inputs

GIB = 1 << 30


def listed():
    return [
        # a short file: the cost of the call itself (the paper's smallest, padded to whole blocks)
        {"name": "ecb_enc_1216", "path": "ecb", "keybits": 128, "decrypt": False, "nbytes": 1216, "in_place": False},
        # the paper's largest file, decrypted under the longest key
        {"name": "ecb_dec_1190416", "path": "ecb", "keybits": 256, "decrypt": True, "nbytes": 1190416,
         "in_place": False},
        # a medium buffer encrypted where it lies
        {"name": "ecb_enc_16mib", "path": "ecb", "keybits": 192, "decrypt": False, "nbytes": 16 << 20,
         "in_place": True},
        # the benchmark's headline buffer
        {"name": "ecb_enc_1gib", "path": "ecb", "keybits": 128, "decrypt": False, "nbytes": GIB, "in_place": False},
        # a record of odd length inside a stream
        {"name": "ctr_18602", "path": "ctr", "keybits": 256, "nbytes": 18602, "block_offset": 77},
        # a large stream that starts and ends off any boundary
        {"name": "ctr_256mib", "path": "ctr", "keybits": 128, "nbytes": (256 << 20) + 5, "block_offset": 1000003},
        # one long CBC message read back
        {"name": "cbc_dec_64mib", "path": "cbc_dec", "keybits": 256, "nbytes": 64 << 20},
        # a disk image sealed page by page: the benchmark's message set
        {"name": "cbc_enc_pages", "path": "cbc_msgs", "keybits": 128, "decrypt": False, "nmsgs": 1 << 18,
         "blocks": 256, "ragged": False, "layout": 1},
        # a thousand files of 64 KiB: few chains, so the latency of a chain counts
        {"name": "cbc_enc_files", "path": "cbc_msgs", "keybits": 256, "decrypt": False, "nmsgs": 1024,
         "blocks": 4096, "ragged": False, "layout": 1},
        # packet-sized messages of mixed length (up to 1.5 KB) opened together
        {"name": "cbc_dec_packets", "path": "cbc_msgs", "keybits": 128, "decrypt": True, "nmsgs": 1 << 16,
         "blocks": 96, "ragged": True, "layout": 1},
        # the batched mix: message lengths 16 B ... 8 MiB, all key sizes, both directions
        {"name": "batch_mix", "path": "batch", "nmsgs": 2000, "hi_bytes": 8 << 20, "layout": 1},
        # host file in, host file out, ordinary (pageable) memory
        {"name": "host_file_1190416", "path": "host", "keybits": 128, "decrypt": False, "nbytes": 1190416},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    path = rng.choice(["ecb", "ecb", "ctr", "cbc_dec", "cbc_msgs", "cbc_msgs", "batch", "host"])
    keybits = rng.choice([128, 192, 256])
    decrypt = rng.random() < 0.5
    if path == "ecb":
        return {"path": path, "keybits": keybits, "decrypt": decrypt, "nbytes": 16 * _log_int(rng, 1, GIB // 16),
                "in_place": rng.random() < 0.25}
    if path == "ctr":
        return {"path": path, "keybits": keybits, "nbytes": _log_int(rng, 1, GIB),
                "block_offset": rng.choice([0, rng.randrange(1 << 32)])}
    if path == "cbc_dec":
        return {"path": path, "keybits": keybits, "nbytes": 16 * _log_int(rng, 1, GIB // 16)}
    if path == "cbc_msgs":
        blocks = _log_int(rng, 4, 4096)
        return {"path": path, "keybits": keybits, "decrypt": decrypt,
                "nmsgs": _log_int(rng, 16, min(1 << 18, GIB // 16 // blocks)), "blocks": blocks,
                "ragged": rng.random() < 0.5, "layout": rng.randrange(1 << 20)}
    if path == "batch":
        return {"path": path, "nmsgs": _log_int(rng, 8, 2000), "hi_bytes": _log_int(rng, 256, 8 << 20),
                "layout": rng.randrange(1 << 20)}
    return {"path": path, "keybits": keybits, "decrypt": decrypt, "nbytes": 16 * _log_int(rng, 1, (16 << 20) // 16)}


def _key(seed, keybits):
    return aes.expand_key(inputs.random_key(seed, keybits))


def _iv(seed):
    return inputs.random_bytes(seed + 1, 16).tobytes()


@functools.lru_cache(maxsize=None)
def _host_pipe():
    return aes.HostPipe()  # a program keeps one


def prepare(case, seed):
    path = case["path"]
    s = {"path": path}
    # the lengths of a message set belong to the case, its bytes, keys and
    # initialisation vectors to the seed
    if path == "batch":
        mix = inputs.message_mix(case["layout"], case["nmsgs"], hi_bytes=case["hi_bytes"])
        keys = [inputs.random_key(seed + int(k), int(b)) for k, b in zip(mix.key_seed, mix.keybits)]
        x = inputs.device_random_bytes(seed, 16 * mix.total_blocks)
        # work items and kernel shape of the benchmark's batched section
        s["batch"] = batch.prepare(batch.messages_from_mix(mix), batch.key_table(keys), x, torch.empty_like(x),
                                   chunk_blocks=2048, cfg=aes.BatchConfig(bpt=4, wg=1024))
        return s
    s["ks"] = _key(seed, case["keybits"])
    s["decrypt"] = case.get("decrypt", False)
    if path == "cbc_msgs":
        make = inputs.cbc_message_set if case["ragged"] else inputs.cbc_equal_messages
        sets = make(case["layout"], case["nmsgs"], case["blocks"])
        recs = np.zeros(len(sets), dtype=aes.CBC_MSG_DTYPE)
        recs["in_block"], recs["out_block"], recs["nblocks"] = sets.in_block, sets.out_block, sets.nblocks
        recs["iv"] = inputs.random_bytes(seed, sets.iv.size).reshape(sets.iv.shape)
        s["msgs"] = torch.from_numpy(recs.view(np.uint8)).to("cuda")
        s["x"] = inputs.device_random_bytes(seed, 16 * sets.in_blocks)
        s["out"] = torch.zeros(16 * sets.out_blocks, dtype=torch.uint8, device="cuda")  # gaps stay zero
        return s
    if path == "host":
        s["x"] = inputs.random_bytes(seed, case["nbytes"])
        s["out"] = np.empty_like(s["x"])
        s["pipe"] = _host_pipe()
        s["op"] = aes.AES_PIPE_ECB_DECRYPT if s["decrypt"] else aes.AES_PIPE_ECB_ENCRYPT
        return s
    s["x"] = inputs.device_random_bytes(seed, case["nbytes"])
    # in place, every pass works on the bytes that the last one left; so the
    # ordinary case writes to a buffer of its own
    s["out"] = s["x"] if case.get("in_place") else torch.empty_like(s["x"])
    if path in ("ctr", "cbc_dec"):
        s["iv"] = _iv(seed)
        s["block_offset"] = case.get("block_offset", 0)
    return s


def run(s):
    path = s["path"]
    if path == "ecb":
        f = aes.ecb_decrypt if s["decrypt"] else aes.ecb_encrypt
        return f(s["ks"], s["x"], out=s["out"])
    if path == "ctr":
        return aes.ctr_crypt(s["ks"], s["iv"], s["x"], out=s["out"], block_offset=s["block_offset"])
    if path == "cbc_dec":
        return aes.cbc_decrypt(s["ks"], s["iv"], s["x"], out=s["out"])
    if path == "cbc_msgs":
        f = aes.cbc_decrypt_msgs if s["decrypt"] else aes.cbc_encrypt_msgs
        return f(s["ks"], s["msgs"], s["x"], out=s["out"])
    if path == "batch":
        s["batch"].launch()
        return s["batch"].out_arena
    return s["pipe"].run(s["op"], s["ks"], s["x"], out=s["out"])


def _blocks(case):
    if case["path"] == "cbc_msgs":
        return case["nmsgs"] * case["blocks"] // (2 if case["ragged"] else 1)  # ragged: the mean length
    if case["path"] == "batch":  # mean of a log-uniform length
        lo, hi = 16, case["hi_bytes"]
        return int(case["nmsgs"] * (hi - lo) / np.log(hi / lo) / 16)
    return -(-case["nbytes"] // 16)


def work(case):
    """Each block read and written once, and the message records; the cipher is table look-ups, not arithmetic."""
    recs = 48 if case["path"] == "cbc_msgs" else 24 if case["path"] == "batch" else 0
    return {"bytes": 32 * _blocks(case) + recs * case.get("nmsgs", 0), "flops": 0}
