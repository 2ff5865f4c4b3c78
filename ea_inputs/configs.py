"""Workload shapes c1..c5, from a tiny correctness case to full caches of 8 to 14 billion parameter models;
the *_mini variants keep the structure (GQA ratio, head_dim, outliers, dtype) at sizes a CPU
oracle finishes in seconds while still spanning several kernel tiles and a ragged tail."""
from dataclasses import dataclass, replace


@dataclass(frozen=True)
class CacheConfig:
    name: str
    dtype: str            # "f32" | "bf16"  (storage type of Q, K, V)
    batch: int
    layers: int
    n_q_heads: int
    n_kv_heads: int
    head_dim: int
    n: int                # cached tokens per head
    window: int           # number of most recent queries the statistics use
    rope_base: float
    n_outliers: int       # outlier channels per KV head (shared with its query group)
    outlier_offset: float
    keep: float           # kept fraction f = n_keep / n   (ratio r = 1 - f)
    seed: int
    horizon_T: int = 512  # future positions the rotary matrix is averaged over (paper: 512)
    epsilon: float = 0.02  # paper's default; 0 is its needle-in-a-haystack variant

    @property
    def group(self) -> int:
        return self.n_q_heads // self.n_kv_heads

    @property
    def n_keep(self) -> int:
        return int(self.n * self.keep)

    def with_(self, **kw) -> "CacheConfig":
        return replace(self, **kw)


CONFIGS = {
    # 1: tiny fp32 correctness case
    "c1": CacheConfig("c1", "f32", 1, 1, 4, 2, 64, 1024, 64, 1e4, 0, 0.0, 0.5, 1),
    # 2: Llama-3.1-8B-shaped, one layer, 16k tokens
    "c2": CacheConfig("c2", "bf16", 1, 1, 32, 8, 128, 16384, 128, 5e5, 4, 8.0, 0.5, 2),
    # 3: Llama-3.1-8B-shaped full cache, 128k tokens x 32 layers (seed 3000 + layer)
    "c3": CacheConfig("c3", "bf16", 1, 32, 32, 8, 128, 131072, 128, 5e5, 4, 8.0, 0.5, 3000),
    # 4: Gemma3-12B-shaped, d=256, batch 4 (seed 4000 + 48*b + layer), rotary base 1e6, window 128
    "c4": CacheConfig("c4", "bf16", 4, 48, 16, 8, 256, 32768, 128, 1e6, 4, 8.0, 0.5, 4000),
    # 5: decode pass, Qwen-14B-shaped: 4608 cached tokens compressed back to 4096, window 512
    "c5": CacheConfig("c5", "bf16", 1, 48, 40, 8, 128, 4608, 512, 1e6, 4, 8.0, 4096 / 4608, 5000),
}


def get_config(name: str) -> CacheConfig:
    return CONFIGS[name]
