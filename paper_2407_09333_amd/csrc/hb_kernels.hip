// hb_kernels.hip -- fixed-length batch-hashing kernels: one lane per message, in index order.
#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstdlib>
#include <type_traits>

#include "hb_device.hpp"
#include "hb_internal.hpp"

namespace hb {

constexpr int kPlainBlock = 256;

// Lane i hashes message i of a fixed-length batch: it starts at i * fixed_len and is
// fixed_len bytes long.
template <int A, bool MANY>
__device__ __forceinline__ void plain_lane(const uint8_t *__restrict__ msgs, uint64_t n, uint64_t fixed_len,
                                           uint8_t *__restrict__ out, uint32_t stride)
{
    const uint64_t i = uint64_t(xcd_contiguous(blockIdx.x, gridDim.x)) * kPlainBlock + threadIdx.x;
    if (i >= n) return;
    uint32_t s[8];
    hash_message<A, kDefaultBurst<A>, MANY>(msgs + i * fixed_len, fixed_len, s);
    store_digest<A>(out + i * stride, s, stride);
}

// For launches with more than one wave per SIMD, and (k_plain_few) for smaller ones.  (The
// offsets, lengths and filter of a packed form, which hb_ragged.hip hashes, are unused.)
template <int A, bool FIXED>
__global__ __launch_bounds__(kPlainBlock) void k_plain(const uint8_t *__restrict__ msgs, const uint64_t *, const uint64_t *,
                                                       uint64_t n, uint64_t fixed_len, uint8_t *__restrict__ out,
                                                       uint32_t stride, const uint8_t *)
{
    static_assert(FIXED, "packed batches: hb_ragged.hip");
    plain_lane<A, true>(msgs, n, fixed_len, out, stride);
}

template <int A>
__global__ __launch_bounds__(kPlainBlock) void k_plain_few(const uint8_t *__restrict__ msgs, uint64_t n, uint64_t fixed_len,
                                                           uint8_t *__restrict__ out, uint32_t stride)
{
    plain_lane<A, false>(msgs, n, fixed_len, out, stride);
}

// Buffer resource word 3 for raw (unswizzled, unformatted) dword access on gfx9-family
// GPUs, and the cache-policy bit of a non-temporal buffer load.
constexpr int kBufferRsrcWord3 = 0x00020000;
constexpr int kCpolNonTemporal = 2;

// Fixed-length batch with message words staged through LDS (the default for dword-aligned
// fixed-length batches; HB_PLAIN_LDS=0 takes k_plain instead).  Each wave owns 64
// consecutive messages.  Two whole blocks of all 64 go per burst: eight 16-byte loads per
// lane, lane (q, p) of load j taking chunk p ^ q of message 8j + q, so each load instruction
// reads eight whole 128-byte lines; the chunks are written to the wave's LDS slice in that
// order and each lane reads back its own message's 128 bytes, the XOR swizzle putting eight
// consecutive lanes on eight different bank groups.  Messages must start on a dword (msgs
// and msg_len 4-byte aligned); the last one or two blocks and a partial last wave go through
// the per-lane path.  The loads are buffer loads off one wave-uniform base, so they take no
// vector address arithmetic (MD5 issues its compression instructions and almost nothing
// more) and few registers.  Each wave keeps the next burst in flight while it compresses the
// current one.  MD5, bound by its reads, streams with non-temporal loads (every line is read
// once, whole, by one instruction); SHA-1 and SM3, bound by their compression, use cached
// loads.  All three run five waves per SIMD, the most the LDS holds (8 KiB per wave).  On
// 2^20 x 1 KiB the three launches took 1,132 us with the compiler's order of the
// compressions and take 998 us with the shared-SIMD order (hb_issue.hpp).
// PAD: len is a multiple of 64, and `pad` the schedule words of the padding-only last block,
// the same for every message of the batch.
template <int A, bool MANY, bool PAD = false>
__device__ __forceinline__ void plain_lds_wave(const uint8_t *__restrict__ msgs, uint64_t n, uint64_t len,
                                               uint8_t *__restrict__ out, const HB_CONSTANT uint32_t *pad = nullptr)
{
    constexpr bool kStream = A == MD5;  // non-temporal loads
    __shared__ u32x4 slice[kPlainBlock / 64][512];  // per wave: 64 messages x 128 bytes
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u), lane = threadIdx.x % 64u;
    const uint64_t m0 = (uint64_t(xcd_contiguous(blockIdx.x, gridDim.x)) * (kPlainBlock / 64) + wave) * 64u;
    if (m0 >= n) return;
    const uint32_t q = lane / 8u, p = lane % 8u, sw = lane & 7u;
    const uint32_t voff = uint32_t(q * len + (p ^ q) * 16u);  // load j adds 8 j len
    const uint64_t nb = (len + 8u) / 64u + 1u, nfast = len / 64u;
    const uint64_t nburst = m0 + 64u <= n ? nfast / 2u : 0u;  // wave-uniform
    const uint8_t *wbase = msgs + m0 * len;
    u32x4 *mine = slice[wave];
    uint32_t s[8];
    init_state<A>(s);
    // The wave's 64 messages through one buffer resource: base in SGPRs, the lane's 32-bit
    // offset in one VGPR, the burst's and load's offset (k 128 + 8 j len) in an SGPR, so a
    // load costs no vector address arithmetic and the loop keeps no 64-bit addresses.  Its
    // range is the wave's 64 messages, 64 len bytes (< 2^31 for the lengths taken here):
    // the furthest load, burst nburst - 1 of message 63, ends at 63 len + 128 nburst <= 64 len,
    // and a read past the range would return zeros rather than touch other memory.  Only
    // whole waves (m0 + 64 <= n) use it.
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(wbase), 0, int(64u * uint32_t(len)), kBufferRsrcWord3);
    auto load = [&](u32x4 *pre, uint64_t k) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            pre[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff, uint32_t(k * 128u + uint64_t(8 * j) * len),
                                                           kStream ? kCpolNonTemporal : 0);
    };
    auto stage = [&](const u32x4 *pre) {
#pragma unroll
        for (int j = 0; j < 8; ++j) mine[j * 64 + lane] = pre[j];
    };
    // The two staged blocks of this lane's message.  MD5 and SHA-1 read both blocks' words
    // from LDS up front, so the second block's reads complete under the first block's
    // compression (16 more registers; SM3, with more state live, reads one block at a time
    // to stay within the registers of five waves per SIMD).
    constexpr bool kReadAhead = A != SM3;
    auto words = [&](int h, uint32_t *w) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4 v = mine[lane * 8u + ((4u * h + i) ^ sw)];
            w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
        }
        if (Traits<A>::kBE)
#pragma unroll
            for (int i = 0; i < 16; ++i) w[i] = bswap32(w[i]);
    };
    auto burst = [&]() {
        if constexpr (kReadAhead) {
            uint32_t w0[16], w1[16];
            // block 0's reads, then block 1's, both before block 0's compression: the wait
            // for block 0 leaves block 1's reads in flight under it
            words(0, w0);
            __builtin_amdgcn_sched_barrier(0);
            words(1, w1);
            __builtin_amdgcn_sched_barrier(0);
            compress<A, MANY>(s, w0);
            compress<A, MANY>(s, w1);
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                uint32_t w[16];
                words(h, w);
                compress<A, MANY>(s, w);
            }
        }
    };
    // A wave's LDS operations complete in order, so a burst's writes to the slice follow the
    // previous burst's reads of it.
    u32x4 pre[8];
    if (nburst) load(pre, 0);
    for (uint64_t k = 0; k < nburst; ++k) {
        stage(pre);
        if (k + 1 < nburst) load(pre, k + 1);
        burst();
    }
    const uint64_t mi = m0 + lane;
    if (mi >= n) return;
    const Msg m = make_msg<A>(msgs + mi * len, len);
    uint64_t blk = nburst * 2u;
    for (; blk < nfast; ++blk) {
        uint32_t w[16];
        load_full_block(m, blk, w);
        compress<A, MANY>(s, w);
    }
    if constexpr (PAD) {
        compress_uniform<A>(s, pad);
    } else if (len % 64u == 0) {
        // the last block is padding only -- 0x80, zeros, the bit length -- and the same for
        // every message of the batch: wave-uniform words, nothing to read or assemble
        constexpr bool kBE = Traits<A>::kBE;
        uint32_t w[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) w[i] = 0u;
        w[0] = kBE ? 0x80000000u : 0x80u;
        const uint64_t bits = len << 3;
        w[14] = kBE ? uint32_t(bits >> 32) : uint32_t(bits);
        w[15] = kBE ? uint32_t(bits) : uint32_t(bits >> 32);
        compress<A, MANY>(s, w);
    } else {
        for (; blk < nb; ++blk) {
            uint32_t w[16];
            load_any_block<Traits<A>::kBE>(m, blk, blk + 1 == nb, w);
            compress<A, MANY>(s, w);
        }
    }
    store_digest<A>(out + mi * Traits<A>::kDigest, s, Traits<A>::kDigest);
}

// For launches with more than one wave per SIMD, and (k_plain_lds_few) for smaller ones.
template <int A>
__global__ __launch_bounds__(kPlainBlock) __attribute__((amdgpu_waves_per_eu(A == MD5 ? 5 : 4))) void
k_plain_lds(const uint8_t *__restrict__ msgs, uint64_t n, uint64_t len, uint8_t *__restrict__ out)
{
    plain_lds_wave<A, true>(msgs, n, len, out);
}

// As k_plain_lds for lengths divisible by 64: the last block's words come formed from the host
// (compress_uniform).  2^22 x 256 bytes, a fifth of whose blocks are such: SM3 602 us with the
// schedule expanded by every lane, 565 so, SHA-1 330 and 310; 300,007 x 64 SM3 21.5 and 20.4.
//
// The kernel's arguments, laid out as a struct's members are: where the words are.
template <int A> struct PadArgs {
    const uint8_t *msgs;
    uint64_t n, len;
    uint8_t *out;
    UniformWords<A> pad;
};

template <int A>
__global__ __launch_bounds__(kPlainBlock) __attribute__((amdgpu_waves_per_eu(A == MD5 ? 5 : 4))) void
k_plain_lds_pad(const uint8_t *__restrict__ msgs, uint64_t n, uint64_t len, uint8_t *__restrict__ out, UniformWords<A>)
{
    static_assert(std::is_same_v<decltype(&k_plain_lds_pad<A>),
                                 void (*)(decltype(PadArgs<A>::msgs), decltype(PadArgs<A>::n), decltype(PadArgs<A>::len),
                                          decltype(PadArgs<A>::out), decltype(PadArgs<A>::pad))>);
    const HB_CONSTANT uint32_t *pad =
        (const HB_CONSTANT uint32_t *)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(PadArgs<A>, pad) / sizeof(uint32_t);
    plain_lds_wave<A, true, true>(msgs, n, len, out, pad);
}

template <int A>
__global__ __launch_bounds__(kPlainBlock) __attribute__((amdgpu_waves_per_eu(A == MD5 ? 5 : 4))) void
k_plain_lds_few(const uint8_t *__restrict__ msgs, uint64_t n, uint64_t len, uint8_t *__restrict__ out)
{
    plain_lds_wave<A, false>(msgs, n, len, out);
}

// The paper's workload (Sec. V-A.2): message i is the 9-character decimal text of
// start + i, zero-padded ("000000000" .. "999999999").  The text is produced in registers,
// so a 9-byte message is one padded block: 9 bytes, 0x80, zeros, bit length 72.
//
// What bounds it: the compression.  The 64 numbers of a wave run over at most one hundreds
// boundary, so their upper seven digits are one of two wave-uniform texts, formed on the
// scalar unit; a lane selects one and forms its last two digits, 12 vector instructions
// where nine divisions by ten of its own took about 60, eight of them quarter-rate multiplies
// (SHA-1 of 10^8 numbers: 1,407 and 1,313 us).
//
// The words of the seven digits of u (u < 10^7): four in the first, three in the second.
template <bool BE> __device__ __forceinline__ void text7(uint32_t u, uint32_t &w0, uint32_t &w1)
{
    uint32_t d[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) {
        const uint32_t q = u / 10u;
        d[k] = 0x30u + (u - q * 10u);
        u = q;
    }
    w0 = BE ? (d[0] << 24) | (d[1] << 16) | (d[2] << 8) | d[3] : d[0] | (d[1] << 8) | (d[2] << 16) | (d[3] << 24);
    w1 = BE ? (d[4] << 24) | (d[5] << 16) | (d[6] << 8) : d[4] | (d[5] << 8) | (d[6] << 16);
}

template <int A, bool MANY>
__global__ __launch_bounds__(kPlainBlock) void k_digits9(uint64_t start, uint64_t n, uint8_t *__restrict__ out)
{
    constexpr bool kBE = Traits<A>::kBE;
    const uint64_t i0 = uint64_t(blockIdx.x) * kPlainBlock + __builtin_amdgcn_readfirstlane(threadIdx.x) / 64u * 64u;
    const uint64_t i = uint64_t(blockIdx.x) * kPlainBlock + threadIdx.x;
    if (i >= n) return;
    const uint32_t v0 = uint32_t(start + i0), u = v0 / 100u;  // wave-uniform; v0 + 63 < 10^9 + 64
    uint32_t a0, a1, b0, b1;
    text7<kBE>(u, a0, a1);
    text7<kBE>(u + 1u, b0, b1);
    const uint32_t r = v0 - u * 100u + threadIdx.x % 64u;  // 0 .. 162
    const bool over = r >= 100u;
    const uint32_t low = over ? r - 100u : r;
    const uint32_t tens = __umul24(low, 103u) >> 10, ones = low - __umul24(tens, 10u);  // low < 100
    uint32_t w[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) w[k] = 0u;
    w[0] = over ? b0 : a0;
    w[1] = over ? b1 : a1;
    if (kBE) {
        w[1] |= 0x30u + tens;
        w[2] = (ones << 24) + 0x30800000u;
        w[15] = 72u;
    } else {
        w[1] |= (tens << 24) + 0x30000000u;
        w[2] = ones + 0x8030u;
        w[14] = 72u;
    }
    uint32_t s[8];
    init_state<A>(s);
    compress<A, MANY>(s, w);
    store_digest<A>(out + i * Traits<A>::kDigest, s, Traits<A>::kDigest);
}

// Byte copy between device-accessible buffers (device memory or the device mapping of
// pinned host memory): 16 bytes per lane per step when both ends are 16-byte aligned.
template <bool VEC>
__global__ __launch_bounds__(256) void k_copy(uint8_t *dst, const uint8_t *src, uint64_t n)
{
    const uint64_t t = uint64_t(blockIdx.x) * 256u + threadIdx.x, step = uint64_t(gridDim.x) * 256u;
    uint64_t head = 0;
    if constexpr (VEC) {
        const uint64_t nv = n / 16u;
        for (uint64_t i = t; i < nv; i += step)
            reinterpret_cast<u32x4 *>(dst)[i] = reinterpret_cast<const u32x4 *>(src)[i];
        head = nv * 16u;
    }
    for (uint64_t i = head + t; i < n; i += step) dst[i] = src[i];
}

hipError_t launch_copy(void *dst, const void *src, uint64_t bytes, hipStream_t stream)
{
    if (bytes == 0) return hipSuccess;
    const bool vec = ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15u) == 0;
    const uint64_t units = vec ? (bytes + 15u) / 16u : bytes;
    const unsigned blocks = unsigned(std::min<uint64_t>((units + 255u) / 256u, 2048u));
    if (vec)
        hipLaunchKernelGGL(k_copy<true>, dim3(blocks), dim3(256), 0, stream, static_cast<uint8_t *>(dst),
                           static_cast<const uint8_t *>(src), bytes);
    else
        hipLaunchKernelGGL(k_copy<false>, dim3(blocks), dim3(256), 0, stream, static_cast<uint8_t *>(dst),
                           static_cast<const uint8_t *>(src), bytes);
    return hipGetLastError();
}

hipError_t launch_digits9(int algo, uint64_t start, uint64_t n, uint8_t *out, hipStream_t stream)
{
    const uint64_t blocks = (n + kPlainBlock - 1) / kPlainBlock;
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const dim3 grid{uint32_t(blocks), 1, 1}, block{kPlainBlock, 1, 1};
    const bool few = few_waves(n);
    switch (algo) {
    case MD5: hipLaunchKernelGGL((few ? k_digits9<MD5, false> : k_digits9<MD5, true>), grid, block, 0, stream, start, n, out); break;
    case SHA1: hipLaunchKernelGGL((few ? k_digits9<SHA1, false> : k_digits9<SHA1, true>), grid, block, 0, stream, start, n, out); break;
    case SM3: hipLaunchKernelGGL((few ? k_digits9<SM3, false> : k_digits9<SM3, true>), grid, block, 0, stream, start, n, out); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// SIMDs of the current device (four per CU), looked up once per device.
uint32_t device_simds()
{
    static std::atomic<uint32_t> cached[64];
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1024;
    uint32_t simds = cached[dev].load(std::memory_order_relaxed);
    if (simds) return simds;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 1024;
    simds = uint32_t(cus) * 4u;
    cached[dev].store(simds, std::memory_order_relaxed);
    return simds;
}

bool few_waves(uint64_t n) { return (n + 63u) / 64u <= device_simds(); }

template <int A>
static hipError_t launch_a(const uint8_t *msgs, uint64_t n, uint64_t fixed_len, uint8_t *out, uint32_t stride,
                           hipStream_t stream)
{
    const uint64_t blocks = (n + kPlainBlock - 1) / kPlainBlock;
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const dim3 grid{uint32_t(blocks), 1, 1}, block{kPlainBlock, 1, 1};
    if (few_waves(n)) hipLaunchKernelGGL(k_plain_few<A>, grid, block, 0, stream, msgs, n, fixed_len, out, stride);
    else hipLaunchKernelGGL((k_plain<A, true>), grid, block, 0, stream, msgs, nullptr, nullptr, n, fixed_len, out, stride, nullptr);
    return hipGetLastError();
}

// Schedule words of the padding-only block of a message of len bytes (RFC 1321 Sec. 3.1-3.2,
// FIPS 180-4 Sec. 5.1.1 and 6.1.2, GB/T 32905 Sec. 5.2-5.3.2).
template <int A> static UniformWords<A> pad_words(uint64_t len)
{
    UniformWords<A> u;
    uint32_t W[80] = {};
    const uint64_t bits = len << 3;
    auto rol = [](uint32_t x, int s) { return (x << s) | (x >> (32 - s)); };
    W[0] = A == MD5 ? 0x80u : 0x80000000u;
    W[14] = A == MD5 ? uint32_t(bits) : uint32_t(bits >> 32);
    W[15] = A == MD5 ? uint32_t(bits >> 32) : uint32_t(bits);
    if constexpr (A == MD5) {
        for (int i = 0; i < 64; ++i) {
            const int j = i & 15;
            u.w[i] = W[i < 16 ? j : (i < 32 ? (1 + 5 * j) & 15 : (i < 48 ? (5 + 3 * j) & 15 : (7 * j) & 15))] + kMd5T[i];
        }
    } else if constexpr (A == SHA1) {
        for (int t = 0; t < 80; ++t) {
            if (t >= 16) W[t] = rol(W[t - 3] ^ W[t - 8] ^ W[t - 14] ^ W[t - 16], 1);
            u.w[t] = W[t] + (t < 20 ? 0x5a827999u : (t < 40 ? 0x6ed9eba1u : (t < 60 ? 0x8f1bbcdcu : 0xca62c1d6u)));
        }
    } else {
        for (int i = 16; i < 68; ++i) {
            const uint32_t x = W[i - 16] ^ W[i - 9] ^ rol(W[i - 3], 15);
            W[i] = x ^ rol(x, 15) ^ rol(x, 23) ^ rol(W[i - 13], 7) ^ W[i - 6];
        }
        for (int j = 0; j < 64; ++j) {
            u.w[j] = W[j] ^ W[j + 4];
            u.w[64 + j] = W[j];
        }
    }
    return u;
}

template <int A>
static hipError_t launch_lds_a(const uint8_t *msgs, uint64_t n, uint64_t len, uint8_t *out, hipStream_t stream)
{
    const uint64_t blocks = (n + kPlainBlock - 1) / kPlainBlock;
    if (blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
    const dim3 grid{uint32_t(blocks), 1, 1}, block{kPlainBlock, 1, 1};
    if (few_waves(n)) hipLaunchKernelGGL(k_plain_lds_few<A>, grid, block, 0, stream, msgs, n, len, out);
    else if (len % 64u == 0) hipLaunchKernelGGL(k_plain_lds_pad<A>, grid, block, 0, stream, msgs, n, len, out, pad_words<A>(len));
    else hipLaunchKernelGGL(k_plain_lds<A>, grid, block, 0, stream, msgs, n, len, out);
    return hipGetLastError();
}

bool plain_lds_applies(const uint8_t *msgs, uint64_t fixed_len, uint32_t stride, int algo)
{
    // all three algorithms by default; HB_PLAIN_LDS=0 keeps them per lane
    const char *v = std::getenv("HB_PLAIN_LDS");
    if (v && std::atoi(v) == 0) return false;
    // dword-aligned messages; 64 messages' offsets fit the loads' 32-bit offsets; packed digests
    return (reinterpret_cast<uintptr_t>(msgs) & 3u) == 0 && fixed_len % 4u == 0 && fixed_len > 0 &&
           fixed_len < (1ull << 25) && stride == uint32_t(digest_size(algo));
}

hipError_t launch_fixed(int algo, const uint8_t *msgs, uint64_t n, uint64_t fixed_len, uint8_t *out, uint32_t stride,
                        hipStream_t stream)
{
    // few messages: chain pairs, unless HB_PLAIN_LDS asks for one of the kernels here
    const bool staged = plain_lds_applies(msgs, fixed_len, stride, algo);
    if (!std::getenv("HB_PLAIN_LDS") && stride == uint32_t(digest_size(algo)) && fixed_chain_applies(algo, n, fixed_len, staged))
        return launch_fixed_chain(algo, msgs, n, fixed_len, out, stream);
    if (staged) {
        switch (algo) {
        case MD5: return launch_lds_a<MD5>(msgs, n, fixed_len, out, stream);
        case SHA1: return launch_lds_a<SHA1>(msgs, n, fixed_len, out, stream);
        case SM3: return launch_lds_a<SM3>(msgs, n, fixed_len, out, stream);
        default: return hipErrorInvalidValue;
        }
    }
    switch (algo) {
    case MD5: return launch_a<MD5>(msgs, n, fixed_len, out, stride, stream);
    case SHA1: return launch_a<SHA1>(msgs, n, fixed_len, out, stride, stream);
    case SM3: return launch_a<SM3>(msgs, n, fixed_len, out, stride, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hb
