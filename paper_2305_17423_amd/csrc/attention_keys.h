// Which keys a thread of the attention kernels reads for its slot of a key block.  Plain C++ (constexpr: host and device), so that
// a host program can hold the same expressions against the bounds of the buffers.  Internal.
#pragma once

namespace fise {

constexpr int AT_BKV = 64;        // keys per block

// A slot holds key `key` (K tile) or the eight keys from `key` on (V^T tile, `key` a multiple of 8) of every block; its
// pointer names them in block 0, and a block of existing keys is read `k0` keys further on.  Where the last block is
// partial (`last`: its last existing key) a slot past the end reads the last existing key, or the last chunk of eight that
// holds an existing one, instead: it steps back from its OWN place, so the read stays inside its row in block 0 as in any other.
// The last chunk may run past n_keys, never past n_keys rounded up to 8, and a V^T row has n_stride >= that many elements.
constexpr int at_key_shift(int k0, int last, int key) { return k0 + (last < key ? last - key : 0); }
constexpr int at_value_shift(int k0, int last, int key) { return at_key_shift(k0, last & ~7, key); }

// ---- attention_turns_kernel: turns of 64 keys (wide heads: 32), brought into LDS by loads of 64 pieces of 16 bytes.  D: the head dim.
template <int D> struct AtTile {
    static constexpr int KD = (D + 15) / 16, DB = (D + 31) / 32, NB = KD <= 5 ? 2 : 1, BK = 32 * NB;      // 16-wide steps and 32-row blocks of the head dim, 32-key blocks and keys of a turn
    // Pieces of 16 bytes of a key's and of a value row in LDS.  Odd numbers: sixteen rows meet no bank twice (value rows of wider heads, which leave no
    // room for that, are swizzled).
    static constexpr int PITCH = D / 8 | 1, VPITCH = KD <= 3 ? 4 * NB + 1 : 4 * NB;
    static constexpr int swizzle(int r) { return NB == 2 ? r >> 1 & 7 : r >> 2 & 3; }          // slot p of a value row holds piece p ^ swizzle
    static constexpr int KL = (BK * PITCH + 63) / 64, VL = (D * VPITCH + 63) / 64;             // loads of 64 pieces of a turn's keys, values
    static constexpr int KB = KL * 1024, VB = VL * 1024, LPW = (KL + VL + 3) / 4;              // LDS of a turn's keys, values; loads of a wave
    static constexpr int AHEAD = KD <= 3 ? 3 : 2, KR = AHEAD + 1, VR = AHEAD + 2;              // turns whose loads are in flight; ring slots
    // Zeros behind the rings: the head's last 16-wide step where half of it lies past the head, value rows past the head.
    static constexpr int PAD = D % 16, TAIL = D % 32, KEYS = VR * VB, ZERO = KEYS + KR * KB, LDS = ZERO + (TAIL ? 64 * NB : 0);

    // What a lane reads, in bytes from the load's base (head h of the turn's first key; row value_row of the head at that key), `last` the turn's last
    // existing key.  LDS row r of a turn holds key (r & 3) + 4 (r / 8 % 2) + 8 (r / 4 % 2) + 16 (r / 16): a lane's eight scores of a 16-key
    // step are eight consecutive keys, the operand of the second product as they stand.
    static constexpr int low(int a, int b) { return a < b ? a : b; }
    static constexpr unsigned key_offset(int slot, int last, int C) {
        const int r = low(slot / PITCH, BK - 1), c = low(slot % PITCH, D / 8 - 1), key = (r & 3) + 4 * (r >> 3 & 1) + 8 * (r >> 2 & 1) + (r & ~15);
        return (unsigned)((key + at_key_shift(0, last, key)) * C + c * 8) * 2u;
    }
    static constexpr int value_row(int load) { return low(load * 64 / VPITCH, D - 1); }
    static constexpr unsigned value_offset(int load, int lane, int last, int n_stride) {
        const int slot = load * 64 + lane, r = slot / VPITCH, c = slot % VPITCH, key = (VPITCH % 2 ? low(c, 4 * NB - 1) : c ^ swizzle(r)) * 8;
        return (unsigned)(low(r, D - 1) - value_row(load)) * (unsigned)n_stride * 2u + (unsigned)(key + at_value_shift(0, last, key)) * 2u;
    }
};
// Turn that a load reads next, `next` being that of the keys now: they run one turn ahead of the values, of which the first group of loads has none.
// (Past the last one: the last one again.)
constexpr int AT_STAYS = 1 << 30;
constexpr int at_next_turn(bool keys, bool first, int next) { return keys ? next + 1 : first ? AT_STAYS : next; }

// ---- attention_few_kernel: blocks of 32 keys, read through buffer descriptors.  What a lane reads is its own offset behind the descriptor's base,
// with no scalar offset: a load is dropped (zeros) where the lane offset is not below the descriptor's size, and how a scalar offset takes part
// in that comparison, above all one that is past the size by itself, need not be known.  Bytes; h: the head; d: its channels.
constexpr int AF_BKV = 32;
constexpr unsigned AF_OOB = 0x80000000u;      // not below any size: keys x channels and channels x n_stride are below 2^30 elements

// Keys: the descriptor of block sb starts at head h of key 32 sb and ends with the batch element; size zero behind the last block.
constexpr unsigned af_key_base(int C, int h, int d, int sb) { return ((unsigned)(sb * AF_BKV) * (unsigned)C + (unsigned)(h * d)) * 2u; }
constexpr unsigned af_key_size(int n_keys, int C, int h, int d, int sb) {
    return sb * AF_BKV < n_keys ? ((unsigned)(n_keys - sb * AF_BKV) * (unsigned)C - (unsigned)(h * d)) * 2u : 0u;
}
// Segment of eight channels of a key of the block (past the head: nothing).
constexpr unsigned af_key_offset(int key, int seg, int C, int d) { return seg * 8 < d ? (unsigned)(key * C + seg * 8) * 2u : AF_OOB; }

// Values: the descriptor holds the rows (channels) of head h; size zero behind the last block.
constexpr unsigned af_value_size(int n_keys, int n_stride, int d, int sb) { return sb * AF_BKV < n_keys ? (unsigned)d * (unsigned)n_stride * 2u : 0u; }
// Eight keys from 32 sb + first on of row 16 i + r.  Keys past n_keys but inside the row's n_stride, or in the rows behind it, are the caller's to hold
// whatever they like: the kernel replaces them by zeros.
constexpr unsigned af_value_row(int r, int first, int n_stride) { return (unsigned)(r * n_stride + first) * 2u; }
constexpr unsigned af_value_offset(unsigned row, int i, int n_stride, int sb) { return row + (unsigned)(sb * (2 * AF_BKV)) + (unsigned)(i * 32) * (unsigned)n_stride; }

}  // namespace fise
