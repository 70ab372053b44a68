"""Which kernel and plan a call takes: the library's own rules, called on the host.

They are C++ functions of the library that the public header does not declare; the names
are their mangled ones."""
import ctypes

import paper_2608_02947_amd as atf

_lib = ctypes.CDLL(atf.LIB_PATH)
_i32, _i64, _bool = ctypes.c_int32, ctypes.c_int64, ctypes.c_bool


def _rule(name, restype, *argtypes):
    f = getattr(_lib, name)
    f.restype, f.argtypes = restype, argtypes
    return f


_direct = _rule("_ZN3atf13decode_directEiiiilibb", _bool, _i32, _i32, _i32, _i32, _i64, _i32, _bool, _bool)
_cols16 = _rule("_ZN3atf13decode_cols16Eiiiillib", _bool, _i32, _i32, _i32, _i32, _i64, _i64, _i32, _bool)
_plan = _rule("_ZN3atf18decode_plan_splitsEiiillibb", _i32, _i32, _i32, _i32, _i64, _i64, _i32, _bool, _bool)
_room = _rule("_ZN3atf13decode_splitsEiil", _i32, _i32, _i32, _i64)


def heads_per_block(group):
    """Query heads of one decode workgroup: the largest divisor of the group up to 32."""
    return max(c for c in range(1, 33) if group % c == 0)


def decode_cols16(batch, group, h_kv, n_k, q_pos, d, ragged=False, cap=None):
    """Whether the heads are the columns of 16x16 matrix tiles (32x32 otherwise)."""
    n_valid = n_k if ragged else min(n_k, q_pos + 1)
    return _cols16(batch, group * h_kv, h_kv, d, n_valid, cap or n_k, heads_per_block(group), ragged)


def decode_direct(batch, group, h_kv, n_k, q_pos, d, rotate=False, ragged=False, cap=None):
    n_valid = n_k if ragged else min(n_k, q_pos + 1)
    return decode_cols16(batch, group, h_kv, n_k, q_pos, d, ragged, cap) and \
        _direct(batch, group * h_kv, h_kv, d, n_valid, heads_per_block(group), rotate, ragged)


def decode_splits(batch, group, h_kv, n_k, q_pos, d, rotate=False):
    """(splits of a uniform batch, the most its workspace has room for)."""
    n_valid = min(n_k, q_pos + 1)
    cols16 = decode_cols16(batch, group, h_kv, n_k, q_pos, d)
    return (_plan(batch, group * h_kv, h_kv, n_k, n_valid, heads_per_block(group), cols16, rotate),
            _room(batch, h_kv, n_k))


_prefill = _rule("_ZN3atf13prefill_wavesEiiiiiiiPKiib", _i32, _i32, _i32, _i32, _i32, _i32, _i32, _i32,
                 ctypes.c_void_p, _i32, _bool)


def prefill_waves(window, batch, n_q, n_k, q_pos0, group, h_kv, rotate=False, cap=None):
    """4 or 8: waves per row block of prefill_short_kernel; 0: prefill_kernel."""
    table = atf.atf_window_table(window)
    return _prefill(batch, n_q, n_k, q_pos0, h_kv, group, cap or n_k, table.ctypes.data,
                    window.head_dim, rotate)
