// The attention's rules from the lengths and heads of a call to the form of the kernel and its split length.  Plain C++, no HIP: a
// host program can walk them.
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
// 6.4 + k (2.05 + 1.22 C) beyond.  That a few units, a thirty-second at most, have a second one goes unnoticed with splits of 512 tokens
// (260 workgroups: 12.5 us, 13.1 as 130 of 1024), and of 768 where all of those are the short end of a batch's last sequence, which come last in its
// grid (an end of 35 tokens, 264 workgroups: 11.9, as 512 a split 12.5; of 565 tokens, 258: 13.6 and 12.2); not with others: a single
// sequence of 2951 tokens of 66 heads 13.8 as 264 of 768 and 12.1 as 396 of 512, 4 of 19187 in all of 13 heads 14.5 as 260 of 1024 and
// 13.2 of 512, 2 of 16482 of 32 over 4 13.4 as 260 of 256 and 12.0 of 512.  The split of least cost against
// fixed ones of 256, 512 or 1024 tokens: 40000 tokens of 32 over 8 heads 20.1 -> 18.1 us, 16 sequences of
// up to 6000 (44000 in all) 24.0 -> 17.8, of up to 4000 of 32 heads 40.1 -> 30.5; 65536 tokens 21.3 either way.
// Over 330 drawn calls from 131072 pairs on, one to sixteen query heads a cache head, 0.93 to 0.96 of them on average (twelve and sixteen heads 0.955).
inline int kv_split_tokens(const int* lengths, int n, int heads, int cus)
{
    int longest = 0;
    for (int b = 0; b < n; ++b) longest = lengths[b] > longest ? lengths[b] : longest;
    int best = 1;
    long long least = 0;
    for (int c = 1; c <= KV_MOST_BLOCKS; ++c) {
        const long long groups = kv_workgroups(lengths, n, heads, c * KV_BLOCK);
        const int end = (lengths[n - 1] - 1) % (c * KV_BLOCK) + 1;
        const bool spare = c == 2 || (c == 3 && n > 1 && end <= KV_BLOCK && groups <= cus + heads);
        const long long k = groups <= cus + (spare ? cus / 32 : 0) ? 1 : (groups + cus - 1) / cus;
        const long long cost = k == 1 ? 860 + 173 * c : 640 + k * (205 + 122 * c);
        if (c == 1 || cost < least) {
            least = cost;
            best = c;
        }
        if (c * KV_BLOCK >= longest) break;
    }
    return best * KV_BLOCK;
}

constexpr int KV_STREAM_L = 512;  // tokens of a workgroup of the streaming form, 1024 for large calls

// Whether one query head a cache head and 131072 to 655360 pairs go to the streaming form instead of the matrix-core form on splits of
// `tokens`, and on how many tokens a workgroup (0: the matrix-core form).  Its grid has a slot for every split of the longest sequence, and
// all have to hold tokens (those without delay it: 16 sequences of up to 600 tokens, 5318 in all, 32 heads, 17.0 us instead of 14.2).  It is
// the faster one (us, streaming / matrix) up to 262144 pairs
//   with one workgroup a unit                     4 sequences of 2048 tokens, 16 heads, 9.8 / 10.5
// and, where the matrix-core form has more than one,
//   with one split a sequence, 192 tokens of it   16 of 293 tokens, 32 heads, 10.4 / 11.9; of 196, 64 heads, 13.0 / 13.4; of 147 12.0 / 11.9
//   with two, up to two workgroups a unit         16 of 782, 16 heads, 12.1 / 12.6; 8 of 1024, 32 heads, 12.5 / 12.7
//   with three, 2 to 2.7 a unit, not full ones    7 of 1098, 32 heads, 13.4 / 14.2; but 3 of 1489, 64 heads, 14.9 / 14.2
//   with three or four, nearly full ones          4 of 2048, 32 heads, 12.6 / 13.3; of 1563 (a last split of 27 tokens) 12.3 / 12.0
//   for a single sequence                         7500 tokens of 32 heads 12.4 / 12.8, 30625 of 8 13.5 / 13.8
// and beyond with one split of up to 1024 tokens a sequence, 1.6 to 4 workgroups a unit: 10 of 887, 48 heads, 16.3 / 17.3, 15 of 10371 in all, 32
// heads, 15.1 / 16.4, 13 of 5661, 64 heads, 17.5 / 19.5 (85 drawn calls 0.97 of the matrix-core form; the worst 14 of 10766, 40 heads, 19.4 / 18.9); with
// 1.5 workgroups a unit 8 of 7462, 48 heads, 16.9 / 15.9.
// Elsewhere the matrix-core form: one workgroup a unit of 768 tokens against one and a half of 512, 18750 tokens of 8 heads 12.8 / 12.1; batches of
// longer sequences level, 4 of 8192, 8 heads, 13.1 / 12.9.  Both err by 1 to 4e-7 there.
inline int kv_stream_tokens(const int* lengths, int n, int heads, int longest, long long total, int cus, int tokens)
{
    const long long pairs = total * heads;
    if (pairs < 131072 || pairs >= 655360) return 0;
    if (pairs > 262144) return longest <= 2 * KV_STREAM_L && 16 * n * heads >= 25 * cus && n * heads <= 4 * cus ? 2 * KV_STREAM_L : 0;
    const int splits = (longest + KV_STREAM_L - 1) / KV_STREAM_L;
    const long long groups = kv_workgroups(lengths, n, heads, KV_STREAM_L), slots = groups * KV_STREAM_L;
    if (groups != static_cast<long long>(splits) * n * heads) return 0;
    if (groups <= cus + cus / 32) return KV_STREAM_L;
    if (kv_workgroups(lengths, n, heads, tokens) <= cus + cus / 32) return 0;
    bool faster = false;
    if (splits == 1) faster = pairs >= 192 * groups;
    else if (groups <= 2 * cus) faster = n == 1 || splits == 2 || (splits <= 4 && 8 * pairs >= 7 * slots);
    else if (splits == 3) faster = 10 * groups <= 27 * cus && 20 * pairs <= 17 * slots;
    return faster ? KV_STREAM_L : 0;
}

enum class KvForm { at_once, stream, matrix };
struct KvPlan {
    KvForm form;
    int tokens;  // of a workgroup
};
constexpr int KV_MAX_L = 256;  // tokens of a workgroup of the form that issues all loads at once, at most: four per lane group

// workgroups of that form for one sequence: an index per (split, query head), padded to whole groups of 8 * rep (kv_place)
inline long long kv_at_once_groups(int splits, int rep, int H_kv) { return 8LL * rep * ((static_cast<long long>(splits) * H_kv + 7) / 8); }

// forced: the "kv_tokens" option, 0 = automatic; more than KV_MAX_L asks for the matrix-core form.
// The form that issues all loads at once for small calls, 128 tokens per workgroup and from 2048 x 32 (token, query head) pairs on
// 256, else the matrix-core form on splits of the length that kv_split_tokens finds, or the streaming form (kv_stream_tokens).  Where the first
// two meet (us, all at once / matrix):
//   one sequence   with two to four query heads a cache head at 65536 pairs (3000 tokens of 32 over 16 9.7 / 9.1, of 32 over 8 9.4 /
//                  9.4; below, 929 of 64 over 16 8.4 / 8.6), with more or one at 131072 (3000 of 32 over 4 9.5 / 9.7, 4001 of 32 with
//                  the query's rotation 10.4 / 10.5 and 5 % more of a decode step)
//   a batch        from 40960 pairs on (below, 8 sequences of 1183 tokens in all, 32 over 8 heads, 8.5 / 8.6), as soon as the first form has more
//                  than two workgroups a unit, those without tokens and the padding of its grid among them, which ragged and short
//                  sequences have most of (16 sequences of 1618 tokens, 32 over 4 heads, 11.4 / 8.8; of 1489, 32 heads, 11.5 / 9.5; 12 of 1248, 48
//                  over 8, 10.1 / 8.6).  Up to two it depends on the query heads a cache head (230 drawn batches):
//                  more than eight: all at once up to 131072 pairs (2 of 936 tokens, 64 over 4 heads, 8.3 / 10.2; of 1406 9.2 / 10.3)
//                  five to eight:   all at once up to 65536 (4 of 1872, 32 over 4, 8.4 / 9.2; of 2812 9.5 / 9.1)
//                  three or four:   all at once up to 65536 where a sequence is longer than a workgroup of the matrix-core form
//                                   (4 of 1872, 32 over 8, 8.6 / 8.8; 16 of 1664 8.7 / 8.4)
//                  two:             matrix-core form (2 of 1874, 32 over 16, 8.8 / 8.1)
//                  one:             all at once up to 65536 where the matrix-core form, a workgroup for every head, has more than one a
//                                   unit (16 of 1872, 32 heads, 9.1 / 9.6; 8 of 1872 8.9 / 8.5)
// Between 40960 and 131072 pairs the first form errs by 5.6e-7 of the result, the matrix-core form by 2.0e-7 (16 drawn batches).
inline KvPlan kv_plan(const int* lengths, int n, bool batched, int H_q, int H_kv, int cus, int forced)
{
    if (forced != 0) return {forced > KV_MAX_L ? KvForm::matrix : KvForm::at_once, forced};
    const int rep = H_q / H_kv, heads = H_kv * ((rep + 15) / 16);  // sixteen query heads at most per workgroup of the matrix-core form
    long long total = 0;
    int longest = 0;
    for (int b = 0; b < n; ++b) {
        total += lengths[b];
        longest = lengths[b] > longest ? lengths[b] : longest;
    }
    const long long pairs = total * H_q;
    const int few = pairs < 65536 ? 128 : KV_MAX_L;
    bool matrix;
    if (pairs >= 131072) matrix = true;
    else if (!batched) matrix = rep >= 2 && rep <= 4 && pairs >= 65536;
    else if (pairs < 40960) matrix = false;
    else if (n * kv_at_once_groups((longest + few - 1) / few, rep, H_kv) > 2 * cus) matrix = true;
    else if (rep > 8) matrix = false;
    else if (rep == 2 || pairs >= 65536) matrix = true;
    else if (rep == 1) matrix = kv_workgroups(lengths, n, heads, KV_BLOCK) <= cus;
    else matrix = rep <= 4 && longest <= KV_BLOCK;
    if (!matrix) return {KvForm::at_once, few};
    const int tokens = kv_split_tokens(lengths, n, heads, cus);
    const int stream = rep == 1 ? kv_stream_tokens(lengths, n, heads, longest, total, cus, tokens) : 0;
    if (stream != 0) return {KvForm::stream, stream};
    return {KvForm::matrix, tokens};
}

}  // namespace rcp
