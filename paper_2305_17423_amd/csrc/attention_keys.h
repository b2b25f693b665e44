// Which keys a thread of attention_kernel reads for its slot of a key block.  Plain C++ (constexpr: host and device), so that
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

}  // namespace fise
