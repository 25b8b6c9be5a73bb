"""How the library splits a score call, and whether bkv_evict takes its fused
launch, asked of the library itself (its own C++ functions), so that the
cases of a test are known to reach what they are meant for."""
import ctypes

import paper_2609_04971_amd as bkv

_SIZES = ("hctl", "cflags", "tk_hist", "tk_head", "tk_cand", "tk_cnt", "ctl_end", "part_m", "part_z", "lse2", "rows",
          "rmeta", "score_end", "scores", "kept", "evict_end")
_INTS = ("P", "nseg", "R_pad_max", "nch", "kgn", "key_chunk", "nch_ws", "rtg")


class Layout(ctypes.Structure):
    """WsLayout of csrc/internal.h."""
    _fields_ = [(n, ctypes.c_size_t) for n in _SIZES] + [(n, ctypes.c_int) for n in _INTS]

    @property
    def groups(self):
        return self.R_pad_max // (16 * self.rtg) if self.rtg else 0

    @property
    def in_scores(self):
        """The chunk statistics lie where the scores will be."""
        return self.nch > self.nch_ws


def layout(d, mean=False) -> Layout:
    f = bkv.lib()._ZN3bkv9ws_layoutERK8bkv_dimsi
    f.restype, f.argtypes = Layout, [ctypes.POINTER(bkv.Dims), ctypes.c_int]
    return f(ctypes.byref(d), bkv.SCORE_MEAN if mean else 0)


def fuses(d) -> bool:
    f = bkv.lib()._ZN3bkv13evict_fusableERK8bkv_dimsRKNS_8WsLayoutE
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.POINTER(bkv.Dims), ctypes.POINTER(Layout)]
    return f(ctypes.byref(d), ctypes.byref(layout(d)))


# Score calls whose chunks are meant to be as given: B, Hkv, G, D, N, W, C, mean, causal, then row groups, key chunk,
# chunks a head and whether the statistics lie where the scores will be.
CHUNK_CASES = [
    # the longest chunk of one group (1664 keys) full and one key more, with the mask, the mean and both row lengths
    (33, 8, 1, 128, 6656, 88, 8, False, True, 1, 1664, 4, False), (33, 8, 1, 128, 6657, 88, 8, True, False, 1, 1408, 5, False),
    (33, 16, 1, 64, 3328, 80, 16, True, True, 1, 1664, 2, False), (33, 16, 1, 64, 3327, 96, 0, False, False, 1, 1664, 2, False),
    # of several (1152)
    (33, 8, 7, 128, 1152, 64, 16, False, True, 4, 1152, 1, False), (33, 8, 7, 64, 1153, 64, 16, True, False, 4, 640, 2, False),
    (33, 8, 5, 128, 1151, 40, 8, True, True, 2, 1152, 1, False),
    # a layer of few tokens: two chunks, which leave a wave's last 32-key groups or whole waves without keys
    (33, 16, 1, 128, 1664, 8, 4, False, True, 1, 896, 2, False), (33, 16, 1, 128, 1665, 8, 4, True, False, 1, 896, 2, False),
    (33, 16, 1, 64, 1537, 16, 0, False, False, 1, 896, 2, False), (65, 8, 1, 128, 1152, 8, 4, False, True, 1, 1152, 1, False),
    (65, 8, 1, 64, 1153, 8, 4, True, False, 1, 640, 2, False), (16, 8, 4, 128, 4223, 32, 16, False, False, 1, 1152, 4, False),
    # the shortest chunk (256), longer than the head
    (65, 8, 1, 128, 127, 4, 3, False, True, 1, 256, 1, False), (65, 8, 1, 64, 33, 4, 3, True, True, 1, 256, 1, False),
    (1, 2, 2, 128, 511, 8, 4, False, True, 1, 256, 2, False), (1, 2, 4, 128, 2049, 32, 16, False, False, 1, 256, 9, False),
    (1, 2, 4, 128, 1919, 32, 16, True, False, 1, 256, 8, False),
    # shorter chunks than those limits, for a fuller last round: the mean, heads of few rows
    (35, 8, 4, 64, 4148, 128, 8, True, False, 4, 896, 5, False), (19, 8, 1, 64, 3413, 64, 8, True, True, 1, 896, 4, False),
    (23, 4, 1, 64, 5282, 160, 16, True, False, 2, 768, 7, True), (58, 1, 1, 64, 7522, 8, 0, False, False, 1, 768, 10, False),
    # statistics where the scores will be, their room exactly full (two and three groups, one), and the next head's
    # scores one key further
    (1, 2, 4, 128, 4608, 44, 16, False, True, 2, 384, 12, True), (2, 3, 4, 64, 4608, 44, 16, True, False, 2, 384, 12, True),
    (1, 2, 8, 128, 6912, 46, 16, False, False, 3, 768, 9, True), (1, 2, 8, 128, 6913, 46, 16, True, True, 3, 896, 8, True),
    (1, 2, 4, 128, 4609, 44, 16, False, False, 2, 512, 10, True), (3, 4, 1, 128, 46437, 32, 16, False, True, 1, 896, 52, True),
    (3, 3, 5, 64, 9001, 33, 7, True, True, 2, 512, 18, True), (4, 8, 4, 128, 12345, 32, 16, False, True, 1, 896, 14, False),
    (1, 1, 8, 128, 5000, 64, 16, False, True, 4, 1024, 5, False),
]


def chunk_dims(case, N_cap=None):
    B, Hkv, G, D, N, W, C = case[:7]
    return bkv.dims(B=B, Hq=Hkv * G, Hkv=Hkv, D=D, N=N, N_cap=N_cap, W=W, C=C, budget=max(64, W), dtype="bf16")
