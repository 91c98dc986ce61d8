// How decode attention is split into workgroups.  Plain C++ (no HIP types),
// so that host-only tests can include this header.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

namespace wq {
namespace attn {

constexpr int kChunkQuantum = 64;      // tokens: a 16-token block for each of a workgroup's four waves
constexpr int kMaxChunk = 4096;        // tokens of a fixed chunk
constexpr int kMaxWhole = 192;         // tokens that one workgroup takes whole
constexpr int kByLengthChunk = 512;    // fixed chunks from here on follow the lengths instead
constexpr int kMaxSeqsByLength = 1024;
constexpr int kMinUnitChunk = 256;     // tokens
// Block-table entries of a chunk that are kept in LDS: 32 KiB, as a fixed
// chunk's doubled (two chunks can become one by the lengths) at one token a
// page.
constexpr int64_t kMaxChunkPages = 2 * kMaxChunk;

struct Plan {
    int64_t chunk;      // tokens of a fixed chunk
    int64_t splits;     // fixed chunks of the longest sequence: the workspace's size
    int64_t units;      // nonzero: chunks by the lengths, at most this many per kv head
    int64_t max_chunk;  // tokens of the longest chunk
};

// Chunk length: a multiple of 64 tokens that gives the split launch about
// `target_blocks` workgroups (what the chip holds at once, so there is a
// single round of them), at most kMaxChunk tokens; with sequences of at most
// WQ_ATTN_MAX_SEQ_LEN tokens that keeps a sequence within kMaxSplits chunks.
//
// `page_size` bounds the chunks by the lengths only; the fixed chunks, and
// with them the workspace, do not depend on it.
inline Plan make_plan(int64_t seqs, int64_t hq, int64_t hkv, int64_t max_seq_len, int64_t page_size,
                      int64_t target_blocks, bool by_length) {
    const int64_t len = std::max<int64_t>(max_seq_len, 1);
    const int64_t want = std::max<int64_t>(1, target_blocks / (seqs * hkv));  // chunks per sequence
    int64_t chunk = (len + want - 1) / want;
    chunk = (chunk + kChunkQuantum - 1) / kChunkQuantum * kChunkQuantum;
    chunk = std::min<int64_t>(std::max<int64_t>(chunk, kChunkQuantum), kMaxChunk);
    // One workgroup takes a short sequence whole: the second launch would cost
    // more than it saves (24 / 8 heads, one sequence: 192 tokens 6.3 us against
    // 7.2 us, 256 tokens 7.9 against 7.4).
    if (len <= kMaxWhole) chunk = (len + kChunkQuantum - 1) / kChunkQuantum * kChunkQuantum;
    Plan pl{chunk, (len + chunk - 1) / chunk, 0, chunk};
    // Several sequences in chunks of at least kByLengthChunk tokens: chunks
    // follow the lengths (which costs two more round trips), in the same
    // workspace.
    if (seqs > 1 && seqs <= kMaxSeqsByLength && seqs * len <= INT32_MAX / 2 && pl.splits > 1 && chunk >= kByLengthChunk &&
        by_length) {
        const int64_t room = seqs * pl.splits;
        pl.units = room;
        // Six query heads or more take over 256 registers: one workgroup per
        // CU, so no more of them than CUs while that cuts every sequence.
        if (hq / hkv >= 6) {
            pl.units = std::min(room, std::max(2 * seqs, 256 / hkv));
            // The longest chunk grows as the units get fewer; its block-table
            // entries have to fit the LDS (64 / 8 heads, 32 sequences of up to
            // 65536 tokens in pages of one: 64 units would need 279 KB).
            pl.units = std::max(pl.units, std::min(room, seqs + (seqs * len + kMaxChunkPages * page_size - 1) /
                                                                    (kMaxChunkPages * page_size)));
        }
        const int64_t hi = (seqs * len + pl.units - seqs - 1) / (pl.units - seqs);
        pl.max_chunk = (std::max<int64_t>(hi, kMinUnitChunk) + 63) / 64 * 64;
    }
    return pl;
}

// Block-table entries that a chunk can use: it may start inside a page.
inline int64_t chunk_pages(const Plan& pl, int64_t page_size) { return pl.max_chunk / page_size + 2; }

}  // namespace attn
}  // namespace wq
