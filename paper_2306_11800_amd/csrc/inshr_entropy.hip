// Entropy stage of the delta (Sec. 6, "Encoding Delta"), host code outside the timed path: every
// group of the regrouped delta stream is run-length encoded -- a run of r equal values v becomes the
// token -v, followed by the token +r when r > 1 -- and the tokens are Huffman coded, one code per
// group (the groups are encoded separately).
//
// Container (little-endian):
//   header   u32 magic "IDE1", u32 n_groups, u64 n, u32 delta_bits, u32 0
//   group    u64 n_values, u64 n_tokens, u64 payload_bits, u32 n_sym, u32 0,
//            n_sym x { i32 token, u32 code length }   in canonical order (length, then token),
//            ceil(payload_bits / 8) bytes: the codes, most significant code bit first, filling
//            every byte from bit 0 upwards
// A group with one distinct token has code length 0 and no payload: n_tokens fixes the sequence.
//
// Bound by the host's instructions per value and token, so: groups (and chunks of large groups) go
// to several threads, tokens are counted in arrays instead of hash maps, codes are appended to a
// 64-bit accumulator, and the decoder looks 11 bits up at a time and appends several equal values
// in one step. 4 Mi values as 1.15 M tokens, 16 threads of an EPYC host: encoded in 1.0 ms (one thread
// 6.3; a map lookup per token and a loop per bit took 20), decoded in 0.7 ms (one thread 4.7; a step
// per bit took 13).
#include <hip/hip_runtime.h>

#include <sched.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstring>
#include <exception>
#include <memory>
#include <new>
#include <thread>
#include <vector>

#include "../../include/inshr.h"

namespace {

// ---- threads ------------------------------------------------------------------------------------

// Values per chunk of work: a thread's start costs about as much as 32 Ki values take to encode.
constexpr uint64_t CHUNK = 1u << 15;
// Values whose tokens are kept at a time (at most 32 MB of them); a larger group is kept whole, since its
// code is known when all of it has been read.
constexpr uint64_t WINDOW = 1u << 23;
constexpr uint32_t MAX_THREADS = 16;

uint32_t threads_for(uint64_t n)
{
    cpu_set_t set;
    uint32_t cpus = sched_getaffinity(0, sizeof(set), &set) == 0 ? (uint32_t)CPU_COUNT(&set) : 1u;
    cpus = std::min(std::max(cpus, 1u), MAX_THREADS);
    return (uint32_t)std::min<uint64_t>(cpus, n / CHUNK + 1);
}

// The threads of one call: run(items, f) hands item 0, 1, .. to whichever thread is free and
// returns on every thread when all items are done, the last one's once(), too.  When memory runs out
// on one of them, failed() says so and whatever is run afterwards does nothing.
class Team {
public:
    explicit Team(uint32_t n) : size_(n) {}

    // body(thread) on every thread of the team, the calling one among them.  A thread works as soon as it is there: sixteen
    // take 0.2 ms to start, one after the other (by a tree of threads no less, the kernel takes turns).  4 Mi values there and
    // back 1.48 ms, 1.66 with a start for all of them together.
    template <class B> void start(B &&body)
    {
        std::vector<std::thread> th;
        const uint32_t want = size_.load(std::memory_order_relaxed);
        th.reserve(want);
        for (uint32_t t = 1; t < want; t++) {
            try {
                th.emplace_back([&body, t] { body(t); });
            } catch (const std::exception &) { // fewer threads than asked for: the rest do it
                break;
            }
        }
        // (until this thread arrives in its turn, nobody has found the team complete)
        size_.store((uint32_t)th.size() + 1, std::memory_order_relaxed);
        body(0u);
        for (std::thread &t : th) t.join();
    }

    template <class F, class O> void run(uint64_t items, F &&f, O &&once)
    {
        for (;;) {
            const uint64_t i = next_.fetch_add(1, std::memory_order_relaxed);
            if (i >= items) break;
            guard([&] { f(i); });
        }
        const uint32_t turn = turn_.load(std::memory_order_relaxed);
        // (first the arrival, then the size: the team may have become smaller until this thread arrived, and the last one to
        // arrive has to find that; the operands of one == come in no order)
        const uint32_t there = arrived_.fetch_add(1, std::memory_order_acq_rel) + 1;
        if (there == size_.load(std::memory_order_relaxed)) {
            guard(once);
            arrived_.store(0, std::memory_order_relaxed);
            next_.store(0, std::memory_order_relaxed);
            turn_.store(turn + 1, std::memory_order_release);
        } else {
            while (turn_.load(std::memory_order_acquire) == turn) std::this_thread::yield();
        }
    }

    template <class G> void guard(G &&g)
    {
        if (failed()) return;
        try {
            g();
        } catch (const std::exception &) { // (std::bad_alloc)
            failed_.store(true, std::memory_order_relaxed);
        }
    }
    bool failed() const { return failed_.load(std::memory_order_relaxed); }

private:
    std::atomic<uint32_t> size_;
    std::atomic<bool> failed_{false};
    std::atomic<uint64_t> next_{0};
    std::atomic<uint32_t> arrived_{0}, turn_{0};
};

// ---- encoder ------------------------------------------------------------------------------------

// Delta values of a stream: w-bit fields, or one u16 per value, which is read as 16-bit fields
struct ValueReader {
    const uint8_t *bytes;
    uint64_t total; // bytes of it
    uint32_t w;
    // 57 bits from bit `bit` on, and zeros past the end
    uint64_t window(uint64_t bit) const
    {
        const uint64_t at = bit >> 3;
        uint64_t x = 0;
        if (at + 8 <= total) memcpy(&x, bytes + at, 8);
        else if (at < total) memcpy(&x, bytes + at, total - at);
        return x >> (bit & 7u);
    }
};

uint64_t reversed(uint64_t code, uint32_t len)
{
    uint64_t r = 0;
    for (uint32_t b = 0; b < len; b++) r |= ((code >> b) & 1ull) << (len - 1u - b);
    return r;
}

struct Sym {
    int32_t token;
    uint32_t len;
    uint64_t count;
    uint64_t code;
};

// A token as the encoder keeps it: value v is v, a run of r < RUNS is `values` + r, a longer one
// (at most one in RUNS values) LONGER | r. The first two index arrays of counts and codes.
constexpr uint32_t RUNS = 1024, LONGER = 0x80000000u, MAX_RUN = 0x7fffffffu;

// A piece of a group. Runs belong to the chunk in which they start; the length of a chunk's last
// run is known when the chunks after it have been read.
struct Chunk {
    uint32_t group, thread;
    uint64_t lo, hi;
    uint32_t *tok;            // those of all its runs but the last
    uint64_t n_tok;
    uint64_t cnt0, n_cnt;     // of the thread's counts: of these tokens
    uint64_t first_start;     // of its runs; hi: none starts here
    uint64_t last_start, last_len;
    uint32_t last_value;
    uint64_t bit0, bits;      // of the group's payload
    uint8_t head, tail;       // bits of bytes shared with the neighbours
};

struct Group {
    uint64_t lo, hi, n_tokens, payload_bits, at;
    uint32_t chunk0, chunk1, thread;
    uint64_t sym0, n_sym; // of the thread's symbols
};

// A run longer than a token can hold is cut.
template <class F> void run_tokens(uint32_t v, uint64_t r, uint32_t values, F &&f)
{
    while (r) {
        const uint32_t part = (uint32_t)std::min<uint64_t>(r, MAX_RUN);
        f(v);
        if (part > 1) f(part < RUNS ? values + part : LONGER | part);
        r -= part;
    }
}

struct Count {
    uint32_t tok;
    uint64_t count;
};

// What one thread of an encoder works with; tokens, counts and symbols of its chunks and groups
// stay in its arrays.
struct Worker {
    uint32_t values; // that there can be
    static constexpr uint64_t SLAB = 8 * CHUNK;
    std::vector<std::unique_ptr<uint32_t[]>> slabs; // of tokens
    size_t slabs_used = 0;
    uint32_t *slab_at = nullptr;
    uint64_t slab_left = 0;
    std::vector<Count> counts;
    std::vector<Sym> syms;
    std::vector<uint64_t> count; // by token, zero between uses
    std::vector<uint32_t> seen, longer;
    std::vector<uint64_t> weight;
    std::vector<uint32_t> parent, depth;
    struct Code {
        uint64_t bits; // first bit lowest
        uint32_t len;
    };
    std::vector<Code> code;                        // by token, of group `loaded`
    std::vector<std::pair<uint32_t, Code>> longer_code; // ascending
    uint32_t loaded = ~0u;
    std::vector<uint64_t> buf;

    void init(uint32_t w) // width of the fields read
    {
        values = 1u << w;
        count.assign(values + RUNS, 0ull);
    }

    // Gives up the tokens, counts and symbols of the window before (the memory is used again)
    void next_window()
    {
        slabs_used = 0;
        slab_left = 0;
        counts.clear();
        syms.clear();
    }

    // the distinct ones of `longer` with their counts
    template <class F> void drain_longer(F &&f)
    {
        std::sort(longer.begin(), longer.end());
        for (size_t i = 0, j; i < longer.size(); i = j) {
            for (j = i + 1; j < longer.size() && longer[j] == longer[i]; j++) {}
            f(longer[i], (uint64_t)(j - i));
        }
        longer.clear();
    }

    // Room for k more tokens (a chunk's at most); what is in a slab stays where it is
    uint32_t *room(uint64_t k)
    {
        if (slab_left < k) {
            if (slabs_used == slabs.size()) slabs.emplace_back(new uint32_t[SLAB]);
            slab_at = slabs[slabs_used++].get();
            slab_left = SLAB;
        }
        return slab_at;
    }

    // Tokens of the runs that start in the chunk, the last of them excepted, and their counts. The
    // fields of a window (as many W-bit ones as 57 bits hold) that differ from the field before
    // them are found together: a field's top bit is set where the exclusive or is not zero. No
    // branch depends on a value or on the length of a run; with runs of a few values none could
    // be predicted (4 Mi values, 1.15 M tokens, one thread: 4.2 ms with a loop over the set bits,
    // 2.9 ms without).
    template <uint32_t W> void read_runs(const ValueReader &rd, bool first, Chunk &c)
    {
        constexpr uint32_t P = 57u / W, BLOCK = 8;
        constexpr uint64_t F = (1ull << W) - 1ull;
        uint64_t ones = 0;
        for (uint32_t j = 0; j < P; j++) ones |= 1ull << (j * W);
        const uint64_t top = ones << (W - 1), low = top - ones;
        // a group's first value is a start: the field before it is taken to be another value
        uint64_t before = rd.window((first ? c.lo : c.lo - 1) * W) & F;
        if (first) before ^= 1ull;
        uint32_t *t = c.tok;
        uint64_t start = c.hi;
        uint32_t value = 0, at[BLOCK * P + 1]; // starts, counted from c.lo
        for (uint64_t i = c.lo; i < c.hi;) {
            uint32_t m = 0;
            for (uint32_t b = 0; b < BLOCK && i < c.hi; b++, i += P) {
                const uint32_t k = (uint32_t)std::min<uint64_t>(P, c.hi - i), from = (uint32_t)(i - c.lo);
                const uint64_t x = rd.window(i * W), d = x ^ (x << W | before);
                const uint64_t s = (((d & low) + low) | d) & top & ((1ull << (k * W)) - 1ull);
                before = (x >> ((k - 1) * W)) & F;
#pragma unroll
                for (uint32_t j = 0; j < P; j++) {
                    at[m] = from + j;
                    m += (s >> (j * W + W - 1)) & 1u;
                }
            }
            uint32_t s = 0;
            if (start == c.hi && m) { // the first run of the chunk
                start = c.first_start = c.lo + at[0];
                value = (uint32_t)(rd.window(start * W) & F);
                s = 1;
            }
            for (; s < m; s++) {
                const uint64_t next = c.lo + at[s];
                const uint32_t r = (uint32_t)(next - start); // at most CHUNK
                t[0] = value;
                t[1] = r < RUNS ? values + r : LONGER | r;
                t += 1 + (r > 1);
                start = next;
                value = (uint32_t)(rd.window(start * W) & F);
            }
        }
        c.n_tok = (uint64_t)(t - c.tok);
        c.last_start = start;
        c.last_value = value;
    }

    void read_chunk(const ValueReader &rd, uint64_t group_lo, Chunk &c)
    {
        c.tok = room(c.hi - c.lo + 2);
        c.first_start = c.hi;
        const bool first = c.lo == group_lo;
        switch (rd.w) {
#define INSHR_W(W) case W: read_runs<W>(rd, first, c); break;
            INSHR_W(1) INSHR_W(2) INSHR_W(3) INSHR_W(4) INSHR_W(5) INSHR_W(6) INSHR_W(7) INSHR_W(8)
            INSHR_W(9) INSHR_W(10) INSHR_W(11) INSHR_W(12) INSHR_W(13) INSHR_W(14) INSHR_W(15) INSHR_W(16)
#undef INSHR_W
        }
        slab_at += c.n_tok;
        slab_left -= c.n_tok;
        count_tokens(c.tok, c.n_tok);
        c.cnt0 = counts.size();
        for (uint64_t j = 0; j < c.n_tok; j++) {
            const uint32_t x = c.tok[j];
            if (!(x & LONGER) && count[x]) {
                counts.push_back(Count{x, count[x]});
                count[x] = 0;
            }
        }
        drain_longer([&](uint32_t x, uint64_t k) { counts.push_back(Count{x, k}); });
        c.n_cnt = counts.size() - c.cnt0;
    }

    void count_tokens(const uint32_t *t, uint64_t k)
    {
        for (uint64_t j = 0; j < k; j++) {
            if (t[j] & LONGER) longer.push_back(t[j]);
            else count[t[j]]++;
        }
    }

    // The code of a group from the counts of its chunks
    void code_group(Group &gr, Chunk *chunks, const Worker *all)
    {
        uint64_t next = gr.hi;
        auto add = [&](uint32_t x, uint64_t k) {
            if (x & LONGER) {
                longer.insert(longer.end(), k, x);
                return;
            }
            if (!count[x]) seen.push_back(x);
            count[x] += k;
        };
        gr.n_tokens = gr.payload_bits = 0;
        for (uint32_t k = gr.chunk1; k-- > gr.chunk0;) {
            Chunk &c = chunks[k];
            c.last_len = 0;
            if (c.first_start < c.hi) {
                c.last_len = next - c.last_start;
                next = c.first_start;
                run_tokens(c.last_value, c.last_len, values, [&](uint32_t x) {
                    add(x, 1);
                    gr.n_tokens++;
                });
            }
            gr.n_tokens += c.n_tok;
            const Count *cc = all[c.thread].counts.data() + c.cnt0;
            for (uint64_t j = 0; j < c.n_cnt; j++) add(cc[j].tok, cc[j].count);
        }
        gr.sym0 = syms.size();
        for (uint32_t x : seen) {
            syms.push_back(Sym{x < values ? -(int32_t)x : (int32_t)(x - values), 0u, count[x], 0ull});
            count[x] = 0;
        }
        seen.clear();
        drain_longer([&](uint32_t x, uint64_t k) { syms.push_back(Sym{(int32_t)(x & ~LONGER), 0u, k, 0ull}); });
        gr.n_sym = syms.size() - gr.sym0;
        build_code(syms.data() + gr.sym0, gr.n_sym);
        for (uint64_t j = 0; j < gr.n_sym; j++) gr.payload_bits += syms[gr.sym0 + j].count * syms[gr.sym0 + j].len;
    }

    // Huffman code lengths by the two-queue construction on the symbols in ascending (count, token)
    // order (leaves before merged nodes on equal weight), then canonical codes in (length, token)
    // order
    void build_code(Sym *sym, size_t k)
    {
        if (k <= 1) return;
        std::sort(sym, sym + k, [](const Sym &a, const Sym &b) {
            return a.count != b.count ? a.count < b.count : a.token < b.token;
        });
        // nodes 0..k-1 are the leaves, k.. the merged ones in creation order (weights ascending)
        weight.resize(2 * k - 1);
        parent.resize(2 * k - 1);
        depth.resize(2 * k - 1);
        for (size_t i = 0; i < k; i++) weight[i] = sym[i].count;
        size_t leaf = 0, node = k, made = k;
        auto take = [&]() -> size_t {
            if (leaf < k && (node >= made || weight[leaf] <= weight[node])) return leaf++;
            return node++;
        };
        while (made < 2 * k - 1) {
            const size_t a = take(), b = take();
            weight[made] = weight[a] + weight[b];
            parent[a] = parent[b] = (uint32_t)made;
            made++;
        }
        depth[2 * k - 2] = 0;
        for (size_t i = 2 * k - 2; i-- > 0;) depth[i] = depth[parent[i]] + 1u;
        for (size_t i = 0; i < k; i++) sym[i].len = depth[i];
        std::sort(sym, sym + k, [](const Sym &a, const Sym &b) {
            return a.len != b.len ? a.len < b.len : a.token < b.token;
        });
        uint64_t next = 0;
        uint32_t len = sym[0].len;
        for (size_t i = 0; i < k; i++) {
            next <<= (sym[i].len - len);
            len = sym[i].len;
            sym[i].code = next++;
        }
    }

    void load(uint32_t g, const Group &gr, const Worker *all)
    {
        if (g == loaded) return;
        loaded = g;
        code.resize(values + RUNS);
        longer_code.clear();
        const Sym *sym = all[gr.thread].syms.data() + gr.sym0;
        for (uint64_t j = 0; j < gr.n_sym; j++) {
            const Code k{reversed(sym[j].code, sym[j].len), sym[j].len};
            const int32_t t = sym[j].token;
            if (t >= (int32_t)RUNS) longer_code.emplace_back(LONGER | (uint32_t)t, k);
            else code[t <= 0 ? (uint32_t)-t : values + (uint32_t)t] = k;
        }
        std::sort(longer_code.begin(), longer_code.end(),
                  [](const auto &a, const auto &b) { return a.first < b.first; });
    }
    Code of(uint32_t x) const
    {
        if (!(x & LONGER)) return code[x];
        return std::lower_bound(longer_code.begin(), longer_code.end(), x,
                                [](const auto &a, uint32_t t) { return a.first < t; })->second;
    }

    // The chunk's codes from bit c.bit0 of the payload. Bytes that it shares with its neighbours
    // are kept in c.head and c.tail.
    void write_chunk(Chunk &c, uint8_t *payload)
    {
        const uint32_t lead = (uint32_t)(c.bit0 & 7u);
        buf.resize((lead + c.bits) / 64 + 3);
        uint8_t *q = (uint8_t *)buf.data();
        uint64_t acc = 0;
        uint32_t nb = lead; // below 8 between tokens
        auto put = [&](uint64_t bits, uint32_t len) { // len <= 56
            acc |= bits << nb;
            nb += len;
            memcpy(q, &acc, 8);
            q += nb >> 3;
            acc >>= nb & 56u;
            nb &= 7u;
        };
        auto token = [&](uint32_t x) {
            const Code k = of(x);
            if (k.len > 56u) {
                put(k.bits & 0xffffffffull, 32);
                put(k.bits >> 32, k.len - 32);
            } else {
                put(k.bits, k.len);
            }
        };
        for (uint64_t j = 0; j < c.n_tok; j++) token(c.tok[j]);
        run_tokens(c.last_value, c.last_len, values, token);
        memcpy(q, &acc, 8);
        const uint8_t *b = (const uint8_t *)buf.data();
        uint64_t from = 0, to = (lead + c.bits) / 8;
        c.head = c.tail = 0;
        if (to < 1) { // all of it within one byte
            c.tail = b[0];
            return;
        }
        if (lead) c.head = b[from++];
        memcpy(payload + c.bit0 / 8 + from, b + from, to - from);
        if ((lead + c.bits) & 7u) c.tail = b[to];
    }
};

template <class T> void put(uint8_t *&p, T v)
{
    memcpy(p, &v, sizeof(T));
    p += sizeof(T);
}
template <class T> bool get(const uint8_t *&p, const uint8_t *end, T &v)
{
    if ((size_t)(end - p) < sizeof(T)) return false;
    memcpy(&v, p, sizeof(T));
    p += sizeof(T);
    return true;
}

constexpr uint32_t MAGIC = 0x31454449u; // "IDE1"

int encode(const ValueReader &rd, uint64_t n, uint32_t delta_bits, const uint64_t *group_off,
           uint32_t n_groups, uint8_t *out, uint64_t out_cap, uint64_t *out_bytes,
           inshr_entropy_stats *stats)
{
    if (!group_off || !out_bytes || n_groups == 0 || delta_bits < 1 || delta_bits > 16) return INSHR_E_ARG;
    if (group_off[0] != 0 || group_off[n_groups] != n) return INSHR_E_SHAPE;
    for (uint32_t g = 0; g < n_groups; g++)
        if (group_off[g] > group_off[g + 1]) return INSHR_E_SHAPE;
    std::vector<Group> groups(n_groups);
    std::vector<Chunk> chunks;
    chunks.reserve(n_groups + n / CHUNK);
    for (uint32_t g = 0; g < n_groups; g++) {
        Group &gr = groups[g];
        gr.lo = group_off[g], gr.hi = group_off[g + 1];
        gr.chunk0 = (uint32_t)chunks.size();
        for (uint64_t lo = gr.lo; lo < gr.hi; lo += CHUNK) {
            chunks.emplace_back();
            chunks.back().group = g;
            chunks.back().lo = lo, chunks.back().hi = std::min(lo + CHUNK, gr.hi);
        }
        gr.chunk1 = (uint32_t)chunks.size();
    }
    std::vector<uint32_t> windows(1, 0u); // first group of each, and their end
    for (uint32_t g = 0; g < n_groups; g++)
        if (g > windows.back() && group_off[g + 1] - group_off[windows.back()] > WINDOW) windows.push_back(g);
    windows.push_back(n_groups);
    inshr_entropy_stats st;
    memset(&st, 0, sizeof(st));
    uint64_t used = 24;
    auto place = [&](uint32_t g0, uint32_t g1) { // where every group goes
        for (uint32_t g = g0; g < g1; g++) {
            Group &gr = groups[g];
            gr.at = used;
            used += 32 + 8ull * gr.n_sym + (gr.payload_bits + 7) / 8;
            st.n_tokens += gr.n_tokens;
            st.table_bytes += 32 + 8ull * gr.n_sym;
            st.payload_bytes += (gr.payload_bits + 7) / 8;
        }
    };
    const uint32_t n_threads = threads_for(n);
    std::vector<Worker> workers(n_threads);
    Worker *all = workers.data();
    auto head_group = [&](uint32_t g, Worker &me) { // header and table; where its chunks' bits go
        const Group &gr = groups[g];
        uint8_t *p = out + gr.at;
        put<uint64_t>(p, gr.hi - gr.lo);
        put<uint64_t>(p, gr.n_tokens);
        put<uint64_t>(p, gr.payload_bits);
        put<uint32_t>(p, (uint32_t)gr.n_sym);
        put<uint32_t>(p, 0u);
        const Sym *sym = all[gr.thread].syms.data() + gr.sym0;
        for (uint64_t j = 0; j < gr.n_sym; j++) {
            put<int32_t>(p, sym[j].token);
            put<uint32_t>(p, sym[j].len);
        }
        if (gr.chunk1 - gr.chunk0 == 1) {
            chunks[gr.chunk0].bit0 = 0;
            chunks[gr.chunk0].bits = gr.payload_bits;
        } else if (gr.chunk1 > gr.chunk0) {
            me.load(g, gr, all);
            uint64_t bit = 0;
            for (uint32_t k = gr.chunk0; k < gr.chunk1; k++) {
                Chunk &c = chunks[k];
                c.bit0 = bit;
                const Count *cc = all[c.thread].counts.data() + c.cnt0;
                for (uint64_t j = 0; j < c.n_cnt; j++) bit += cc[j].count * me.of(cc[j].tok).len;
                run_tokens(c.last_value, c.last_len, me.values, [&](uint32_t x) { bit += me.of(x).len; });
                c.bits = bit - c.bit0;
            }
        }
    };
    auto payload_of = [&](const Group &gr) { return out + gr.at + 32 + 8ull * gr.n_sym; };
    auto join_bytes = [&](uint32_t g0, uint32_t g1) { // bytes shared by chunks
        for (uint32_t g = g0; g < g1; g++) {
            const Group &gr = groups[g];
            if (!gr.payload_bits) continue;
            uint8_t *p = payload_of(gr);
            for (int pass = 0; pass < 2; pass++)
                for (uint32_t k = gr.chunk0; k < gr.chunk1; k++) {
                    const Chunk &c = chunks[k];
                    const uint64_t end = c.bit0 + c.bits;
                    if (c.bit0 / 8 < end / 8 && (c.bit0 & 7u)) {
                        if (pass) p[c.bit0 / 8] |= c.head;
                        else p[c.bit0 / 8] = 0;
                    }
                    if (end & 7u) {
                        if (pass) p[end / 8] |= c.tail;
                        else p[end / 8] = 0;
                    }
                }
        }
    };

    bool fits = false;
    Team team(n_threads);
    auto none = [] {};
    team.start([&](uint32_t thread) {
        Worker &me = workers[thread];
        team.guard([&] { me.init(rd.w); });
        for (size_t w = 0; w + 1 < windows.size(); w++) {
            const uint32_t g0 = windows[w], g1 = windows[w + 1];
            const uint32_t c0 = groups[g0].chunk0, n_chunks = groups[g1 - 1].chunk1 - c0;
            me.next_window();
            team.run(n_chunks, [&](uint64_t k) {
                Chunk &c = chunks[c0 + k];
                c.thread = thread;
                me.read_chunk(rd, groups[c.group].lo, c);
            }, none);
            team.run(g1 - g0, [&](uint64_t k) {
                Group &gr = groups[g0 + k];
                gr.thread = thread;
                me.code_group(gr, chunks.data(), all);
            }, [&] {
                place(g0, g1);
                fits = out && used <= out_cap;
            });
            if (!fits) continue; // (the sizes of the rest are wanted all the same)
            team.run(g1 - g0, [&](uint64_t k) { head_group((uint32_t)(g0 + k), me); }, none);
            team.run(n_chunks, [&](uint64_t k) {
                Chunk &c = chunks[c0 + k];
                const Group &gr = groups[c.group];
                if (!gr.payload_bits) return;
                me.load(c.group, gr, all);
                me.write_chunk(c, payload_of(gr));
            }, [&] { join_bytes(g0, g1); });
        }
    });
    if (team.failed()) throw std::bad_alloc();
    if (fits) {
        uint8_t *p = out;
        put<uint32_t>(p, MAGIC);
        put<uint32_t>(p, n_groups);
        put<uint64_t>(p, n);
        put<uint32_t>(p, delta_bits);
        put<uint32_t>(p, 0u);
    }
    *out_bytes = used;
    if (stats) *stats = st;
    return fits ? INSHR_OK : INSHR_E_CAPACITY;
}

// ---- decoder ------------------------------------------------------------------------------------

struct Coded { // a group of the container
    uint64_t pos, n_values, n_tokens, payload_bits;
    uint32_t n_sym;
    const uint8_t *table, *payload;
    uint64_t head, tail; // bits of words shared with the neighbours
    bool ok;
};

// Appends w-bit fields from bit `bit` of `packed` on, by way of a small buffer: whole words go to it
// without a branch, and words shared with what lies before or after are kept apart.
struct FieldWriter {
    static constexpr uint32_t WORDS = 512;
    uint64_t *to, acc = 0, head = 0;
    uint32_t nb, at = 0; // bits of acc (below 64 between fields); words in buf
    bool shared;         // the first word in buf is shared with the group before
    uint64_t buf[WORDS + 1];
    FieldWriter(uint64_t *packed, uint64_t bit)
        : to(packed + (bit >> 6)), nb((uint32_t)(bit & 63u)), shared((bit & 63u) != 0) {}
    void put(uint64_t bits, uint32_t len) // len < 64, no bits above len
    {
        buf[at] = acc | bits << nb;
        const uint32_t sum = nb + len;
        const bool full = sum >= 64u;
        acc = full ? (bits >> 1) >> (63u - nb) : buf[at];
        at += full;
        nb = sum & 63u;
        if (at == WORDS) flush();
    }
    void flush()
    {
        uint32_t from = 0;
        if (shared && at) {
            head = buf[0];
            shared = false;
            from = 1;
        }
        memcpy(to + from, buf + from, 8ull * (at - from));
        to += at;
        at = 0;
    }
};

// Bits looked up at once: tokens of a group take 3 to 8 bits, and 2^11 entries stay in the L1 cache.
constexpr uint32_t LOOK = 11;

struct Decoder { // one thread's tables
    // What the next bits stand for: a value, once (one token) or a run of it (two), or, as `again`,
    // more of the value before (one token)
    struct Entry {
        uint32_t run;
        uint16_t value;
        uint8_t len; // 0: a longer code
        uint8_t tokens : 2, again : 1;
    };
    std::vector<Entry> look;
    std::vector<int32_t> token;
    uint64_t first_code[65], count[65];
    uint32_t first_sym[65], look_bits;

    // The canonical code of a group; false: the table is none.  Lengths may name more codes than there
    // are (or be 0): those past the last code of their length stand for nothing.
    bool load(const Coded &c, uint32_t w)
    {
        token.resize(c.n_sym);
        memset(count, 0, sizeof(count));
        uint32_t before = 0;
        const uint8_t *p = c.table, *end = p + 8ull * c.n_sym;
        for (uint32_t i = 0; i < c.n_sym; i++) {
            uint32_t len = 0;
            get(p, end, token[i]);
            get(p, end, len);
            if (len > 63u || (i && len < before)) return false;
            count[len]++;
            before = len;
        }
        look_bits = 0;
        if (c.n_sym <= 1) return true;
        uint64_t code = 0;
        uint32_t s = 0;
        for (uint32_t l = 0; l <= 63; l++) {
            first_code[l] = code;
            first_sym[l] = s;
            code = (code + count[l]) << 1;
            s += (uint32_t)count[l];
        }
        // an entry costs about as much to make as two tokens without it
        while (look_bits < LOOK && (4ull << look_bits) <= c.n_tokens) look_bits++;
        const uint64_t size = 1ull << look_bits;
        look.assign(size, Entry{0, 0, 0, 0, 0});
        for (uint32_t l = 1; l <= look_bits; l++)
            for (uint64_t k = 0; k < count[l] && first_code[l] + k < (1ull << l); k++) {
                const int32_t t = token[first_sym[l] + k];
                Entry e{1u, (uint16_t)(0u - (uint32_t)t), (uint8_t)l, 1, 0}; // (INT32_MIN has no negative)
                if (t > 0) {
                    e.run = (uint32_t)t - 1u;
                    e.again = 1;
                } else if ((uint32_t)(-(int64_t)t) >> w) {
                    continue; // no value: left to the slow path, which refuses it
                }
                for (uint64_t i = reversed(first_code[l] + k, l); i < size; i += 1ull << l) look[i] = e;
            }
        // a value whose run length is among the bits, too
        for (uint64_t i = 0; i < size; i++) {
            Entry &e = look[i];
            if (!e.len || e.again) continue;
            const Entry &r = look[i >> e.len];
            if (r.len && r.again && (uint32_t)e.len + r.len <= look_bits) {
                e.run += r.run;
                e.len += r.len;
                e.tokens = 2;
            }
        }
        return true;
    }

    // the next token from bit `bit` on; false: the payload ends first, or no code is there
    bool next_slow(const Coded &c, uint64_t &bit, int32_t &t) const
    {
        uint64_t code = 0;
        for (uint32_t l = 1; l <= 63u; l++) {
            if (bit >= c.payload_bits) return false;
            code = (code << 1) | ((c.payload[bit >> 3] >> (bit & 7u)) & 1u);
            bit++;
            if (count[l] && code >= first_code[l] && code - first_code[l] < count[l]) {
                t = token[first_sym[l] + (uint32_t)(code - first_code[l])];
                return true;
            }
        }
        return false;
    }

    // the group's runs to run(v, r)
    template <class R> bool group(const Coded &c, uint32_t w, R &&run)
    {
        if (!load(c, w)) return false;
        const uint64_t mask = (1ull << look_bits) - 1, whole = (c.payload_bits + 7) / 8;
        uint64_t bit = 0, done = 0, k = 0;
        uint32_t last = 0;
        bool have_last = false;
        while (k < c.n_tokens) {
            if (look_bits && (bit >> 3) + 8 <= whole) {
                uint64_t x;
                memcpy(&x, c.payload + (bit >> 3), 8);
                const Entry e = look[(x >> (bit & 7u)) & mask];
                if (e.len && e.tokens <= c.n_tokens - k && bit + e.len <= c.payload_bits && e.run <= c.n_values - done &&
                    (have_last || !e.again)) {
                    last = e.again ? last : e.value;
                    have_last = true;
                    bit += e.len;
                    k += e.tokens;
                    done += e.run;
                    run(last, (uint64_t)e.run);
                    continue;
                }
            }
            int32_t t;
            if (c.n_sym == 1) t = token[0];
            else if (!next_slow(c, bit, t)) return false;
            k++;
            if (t <= 0) {
                last = (uint32_t)(-(int64_t)t);
                have_last = true;
                if (last >> w || done >= c.n_values) return false;
                run(last, 1ull);
                done++;
            } else {
                const uint64_t r = (uint64_t)t - 1;
                if (!have_last || r > c.n_values - done) return false;
                run(last, r);
                done += r;
            }
        }
        return done == c.n_values;
    }
};

int decode(const uint8_t *in, uint64_t in_bytes, uint64_t n, uint32_t delta_bits, uint32_t n_groups,
           uint64_t *packed, uint16_t *values, uint64_t *group_off)
{
    const uint8_t *p = in, *end = in + in_bytes;
    uint32_t magic = 0, G = 0, w = 0, zero = 0;
    uint64_t nn = 0;
    if (!get(p, end, magic) || !get(p, end, G) || !get(p, end, nn) || !get(p, end, w) || !get(p, end, zero))
        return INSHR_E_SHAPE;
    if (magic != MAGIC || G != n_groups || nn != n || w != delta_bits || w < 1 || w > 16) return INSHR_E_SHAPE;
    if ((uint64_t)(end - p) / 32 < G) return INSHR_E_SHAPE;
    std::vector<Coded> groups(G);
    uint64_t pos = 0;
    for (uint32_t g = 0; g < G; g++) {
        Coded &c = groups[g];
        c.pos = pos;
        if (!get(p, end, c.n_values) || !get(p, end, c.n_tokens) || !get(p, end, c.payload_bits) ||
            !get(p, end, c.n_sym) || !get(p, end, zero))
            return INSHR_E_SHAPE;
        if (group_off) group_off[g] = pos;
        if (c.n_values > n - pos || (uint64_t)(end - p) < 8ull * c.n_sym) return INSHR_E_SHAPE;
        c.table = p;
        p += 8ull * c.n_sym;
        c.payload = p;
        const uint64_t nbytes = c.payload_bits / 8 + (c.payload_bits % 8 != 0);
        if ((uint64_t)(end - p) < nbytes) return INSHR_E_SHAPE;
        p += nbytes;
        pos += c.n_values;
    }
    if (group_off) group_off[G] = pos;
    if (pos != n) return INSHR_E_SHAPE;

    std::vector<uint32_t> order(G); // a group is one thread's: the longest first
    for (uint32_t g = 0; g < G; g++) order[g] = g;
    std::sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) {
        return groups[a].n_tokens != groups[b].n_tokens ? groups[a].n_tokens > groups[b].n_tokens : a < b;
    });
    Team team(std::min(threads_for(n), std::max(G, 1u)));
    const uint32_t per = 63u / w; // fields appended in one step
    uint64_t ones = 0;
    for (uint32_t i = 0; i < per; i++) ones |= 1ull << (i * w);
    team.start([&](uint32_t) {
        Decoder dec;
        team.run(G, [&](uint64_t i) {
            Coded &c = groups[order[i]];
            if (values) {
                uint16_t *to = values + c.pos;
                c.ok = dec.group(c, w, [&](uint32_t v, uint64_t r) { to = std::fill_n(to, r, (uint16_t)v); });
                return;
            }
            FieldWriter fw(packed, c.pos * w);
            c.ok = dec.group(c, w, [&](uint32_t v, uint64_t r) {
                const uint64_t many = v * ones;
                for (; r > per; r -= per) fw.put(many, per * w);
                fw.put(many & ((1ull << (r * w)) - 1ull), (uint32_t)r * w);
            });
            fw.flush();
            c.head = fw.head;
            c.tail = fw.acc;
        }, [] {});
    });
    if (team.failed()) throw std::bad_alloc();
    for (const Coded &c : groups)
        if (!c.ok) return INSHR_E_SHAPE;
    if (packed)
        for (int pass = 0; pass < 2; pass++) // words shared by groups
            for (const Coded &c : groups) {
                const uint64_t from = c.pos * w, to = (c.pos + c.n_values) * w;
                if (from / 64 < to / 64 && (from & 63u)) {
                    if (pass) packed[from / 64] |= c.head;
                    else packed[from / 64] = 0;
                }
                if (from < to && (to & 63u)) {
                    if (pass) packed[to / 64] |= c.tail;
                    else packed[to / 64] = 0;
                }
            }
    return INSHR_OK;
}

} // namespace

extern "C" {

int inshr_entropy_encode(const uint64_t *packed, const uint16_t *values, uint64_t n,
                         uint32_t delta_bits, const uint64_t *group_off, uint32_t n_groups,
                         uint8_t *out, uint64_t out_cap, uint64_t *out_bytes,
                         inshr_entropy_stats *stats)
{
    if ((packed == nullptr) == (values == nullptr)) return INSHR_E_ARG; // exactly one of the two
    const ValueReader rd = packed ? ValueReader{(const uint8_t *)packed, ((n * delta_bits + 63) / 64) * 8, delta_bits}
                                  : ValueReader{(const uint8_t *)values, 2 * n, 16u};
    try {
        return encode(rd, n, delta_bits, group_off, n_groups, out, out_cap, out_bytes, stats);
    } catch (const std::exception &) { // (std::bad_alloc)
        *out_bytes = 0; // (not NULL: checked before anything is allocated)
        return INSHR_E_CAPACITY;
    }
}

int inshr_entropy_decode(const uint8_t *in, uint64_t in_bytes, uint64_t n, uint32_t delta_bits,
                         uint32_t n_groups, uint64_t *packed, uint16_t *values, uint64_t *group_off)
{
    if (!in || (packed == nullptr) == (values == nullptr)) return INSHR_E_ARG;
    try {
        return decode(in, in_bytes, n, delta_bits, n_groups, packed, values, group_off);
    } catch (const std::exception &) { // (std::bad_alloc)
        return INSHR_E_CAPACITY;
    }
}

} // extern "C"
