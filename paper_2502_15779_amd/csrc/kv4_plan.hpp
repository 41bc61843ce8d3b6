// The matrix-core attention's rule from the lengths of a call to the split length.  Plain C++, no HIP: a host program can walk it.
#pragma once

namespace rcp {

constexpr int KV_BLOCK = 256;        // tokens that the four wavefronts of a workgroup take at a time, a chunk of 64 each
// Blocks of a split at most.  The rounding of a running sum grows with the tokens a wavefront adds up: 16 sequences of up to 4096
// tokens of 32 heads are off by 3.1e-7 with splits of 1024 and by 5.4e-7 with 2048, which would take 31.3 us instead of 34.5 for
// 131072 tokens of 32 over 8 heads and 17.2 instead of 18.1 (with 1280) for 40000.
constexpr int KV_MOST_BLOCKS = 4;

// workgroups of a call: a split of `tokens` tokens each, for every cache head (and sixteen query heads)
inline long long kv_workgroups(const int* lengths, int n, int heads, int tokens)
{
    long long splits = 0;
    for (int b = 0; b < n; ++b) splits += (lengths[b] + tokens - 1) / tokens;
    return splits * heads;
}

// How long a launch takes is set by the compute unit with the most workgroups, and a workgroup costs its chunks and 1.7 chunks more
// for the query, the merge of its wavefronts and the wait for its first tokens.  Measured over 20 calls (32 over 8, 64 over 8, 32
// over 16 and 64 over 4 heads; one sequence of 5000 to 131072 tokens, ragged batches of 16000 to 65000) with 1 to 16 blocks a split:
// with C blocks a split and k workgroups on the fullest unit a call takes 8.6 + 1.73 C us for k = 1, where every wait shows, and
// 6.4 + k (2.05 + 1.22 C) beyond; that a few units have a second one goes unnoticed up to a thirty-second
// of them (12483 tokens of 32 over 16 heads as 272 workgroups of 768 tokens 14.7 us, as 400 of 512 13.5).  The split of least cost against
// fixed ones of 256, 512 or 1024 tokens: 40000 tokens of 32 over 8 heads 20.1 -> 18.1 us, 16 sequences of
// up to 6000 (44000 in all) 24.0 -> 17.8, of up to 4000 of 32 heads 40.1 -> 30.5; 65536 tokens 21.3 either way.
inline int kv_split_tokens(const int* lengths, int n, int heads, int cus)
{
    int longest = 0;
    for (int b = 0; b < n; ++b) longest = lengths[b] > longest ? lengths[b] : longest;
    int best = 1;
    long long least = 0;
    for (int c = 1; c <= KV_MOST_BLOCKS; ++c) {
        const long long groups = kv_workgroups(lengths, n, heads, c * KV_BLOCK);
        const long long k = groups <= cus + cus / 32 ? 1 : (groups + cus - 1) / cus;
        const long long cost = k == 1 ? 860 + 173 * c : 640 + k * (205 + 122 * c);
        if (c == 1 || cost < least) {
            least = cost;
            best = c;
        }
        if (c * KV_BLOCK >= longest) break;
    }
    return best * KV_BLOCK;
}

}  // namespace rcp
