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
